"""Entries of the work-order file that other kernels wrote are not applied.  A key
that is found returns before any launch, one that is not asks for its workspace
first, so no device is needed."""
import ctypes

import pytest

import paper_1010_5636_amd as ndq

DIMS = (8, 8, 8, 16)
ENTRY = "mrhs 8 8 8 16 1 1 12 6 2 3 1 -1 1 -1 42.5"


def tune():
    nb = ndq.ndq
    g = ndq.Geometry(DIMS)
    links = nb._Gauge(0x1000, ndq.F32, 12)   # never dereferenced
    r = nb._MrhsTuneResult()
    rc = nb.lib().ndq_autotune_mrhs(g.handle, ctypes.byref(links), ndq.F32, 6, 2, 1, None, 0, ctypes.byref(r), None)
    return rc, r.as_dict(), nb.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, 6, 2)


@pytest.mark.parametrize("tag", ["", " v0", " v1", " v1000000", " v", " 2"])
def test_entry_of_other_kernels(tmp_path, monkeypatch, tag):
    cache = tmp_path / "tune.txt"
    cache.write_text(ENTRY + tag + "\n")
    monkeypatch.setenv("NDQ_TUNE_CACHE", str(cache))
    rc, r, order = tune()
    assert rc != 0 and r["cached"] == 0    # asks for a workspace: would time
    assert order["rg"] != 3


def test_entry_of_these_kernels(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    cache.write_text(ENTRY + "\n" + ENTRY.replace("12 6 2 3 1", "12 6 2 2 1") + " v2\n")
    monkeypatch.setenv("NDQ_TUNE_CACHE", str(cache))
    g = ndq.Geometry(DIMS)
    before = ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, 6, 2)
    try:
        rc, r, order = tune()
        assert rc == 0 and r["cached"] == 1 and r["us_best"] == 42.5
        assert (order["rg"], order["group_major"]) == (2, 1)
    finally:
        ndq.ndq.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, 6, 2, **before)
