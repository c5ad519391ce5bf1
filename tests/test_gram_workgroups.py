"""Workgroups of the Gram kernel: no more than run at once where a few more would
take a second round, and never more than the workspace has partial results for.
Called by its C++ name: it is no entry point of the library."""
import ctypes

import pytest

import paper_1010_5636_amd as ndq


def wgs(na, nb, nw):
    f = getattr(ndq.ndq.lib(), "_ZN3ndq8gram_wgsEiii")   # ndq::gram_wgs(int, int, int)
    f.restype = ctypes.c_int
    return f(ctypes.c_int(na), ctypes.c_int(nb), ctypes.c_int(nw))


def most(na, nb):
    """Partial results in 32 MiB, at most 4096."""
    tile = 16 * -(-na // 16) * 16 * -(-nb // 16) * 16
    return min(4096, (32 << 20) // tile)


@pytest.mark.parametrize("na,nb", [(48, 64), (40, 50), (33, 49), (64, 48), (60, 40), (49, 33), (64, 32), (60, 20),
                                   (64, 64), (60, 60), (48, 48), (48, 1), (33, 16)])
def test_one_round_of_two_per_cu(na, nb):
    assert wgs(na, nb, most(na, nb)) == 512


def test_other_blocks_and_small_lattices():
    assert wgs(20, 12, most(20, 12)) == 1024
    assert wgs(1, 1, 4096) == 1024
    assert wgs(60, 12, most(60, 12)) == most(60, 12) == 2048
    for na in range(1, 65):
        for nb in range(1, 65):
            for nw in (1, 2, 100, 511):
                assert wgs(na, nb, nw) == nw
