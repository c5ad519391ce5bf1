"""Replayed multi-shift iterations follow the launch shape in use, its tile order
too: the order says which tile's |out|^2 each partial sum holds, so a replay of
another order adds them up in another sequence than the eager launches do.  The
shape is set by its C++ name, as the autotuner sets it (it picks by time)."""
import ctypes

import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402

DIMS = (8, 8, 8, 16)   # 8 tiles a slice: chunks of 4


def set_order(prec, recon, order):
    """ndq::set_launch_tuning(lattice, sprec, lprec, recon, 2, {block 0, XCD remap, order})."""
    f = getattr(ndq.ndq.lib(), "_ZN3ndq17set_launch_tuningERKNS_5GeomKEiiiiRKNS_6TuningE")
    f.restype = None
    lattice = (ctypes.c_int32 * 64)(*DIMS)   # the extents come first; the rest is not read
    shape = (ctypes.c_int * 3)(0, 1, order)
    f(lattice, ctypes.c_int(prec), ctypes.c_int(prec), ctypes.c_int(recon), ctypes.c_int(2), shape)


@pytest.mark.parametrize("prec,recon,degree,tol", [(ndq.F64, 18, 12, 1e-12), (ndq.F32, 12, 6, 1e-6)])
def test_replays_follow_the_tile_order(prec, recon, degree, tol):
    g = ndq.Geometry(DIMS)
    U = ndq.GaugeField.pack(g, torch.from_numpy(synthetic.gauge_field(DIMS)).cuda(), prec, recon)
    x = ndq.SpinorField.pack(g, torch.from_numpy(synthetic.spinor(g.volume, seed=51)).cuda(), prec, ndq.FULL)
    ap = ndq.Approx(ndq.ZOLOTAREV, 0.08, degree)
    eager, graph = (ndq.Overlap(g, -1.4, ap, 6.6, tol=tol, check_every=4, graph=k) for k in (False, True))
    out = []
    try:
        for order in (0, 1, 0, 1):
            set_order(prec, recon, order)
            ys = []
            for ov in (eager, graph):
                y = x.like()
                ndq.apply_sign(g, U, ov, x, y)
                ys.append(y.buf)
            torch.cuda.synchronize()
            assert torch.equal(ys[0], ys[1]), f"order {order}"
            out.append(ys[0])
    finally:
        ndq.ndq.set_launch_for(prec, prec, recon, 0, True)   # drops the shapes set per lattice
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
