"""The |out|^2 sums that a one-field launch leaves for the multi-shift CG, in every
format and launch shape, without and with extra vectors: the blocks' sums add up to
the norm of the field as stored (the squares are exact in FP64: 1e-13 for the sums
in any order).  Called by the C++ name, as the iteration calls it."""
import ctypes

import numpy as np
import pytest

import synthetic
from oracle import geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402

M = -1.4


class Coef(ctypes.Structure):
    _fields_ = [("f", ctypes.c_double), ("d", ctypes.c_void_p)]


def q_combo(g, U, x, y, vectors):
    """y = 0.7 Q x + sum 0.3 v; the sums of its blocks."""
    lib = ndq.ndq.lib()
    sums = torch.full((g.volume,), np.nan, dtype=torch.float64, device="cuda")
    f = getattr(lib, "_ZN3ndq7q_comboEPK8ndq_geomPK9ndq_gaugedPK10ndq_spinorS8_NS_4CoefEiPKS8_PKS9_PdP12ihipStream_t")
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_double, ctypes.c_void_p, ctypes.c_void_p, Coef,
                  ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    n = len(vectors)
    v = (ctypes.c_void_p * 3)(*[ctypes.addressof(w.desc) for w in vectors])
    c = (Coef * 3)(*[Coef(0.3, None)] * 3)
    rc = f(g.handle, ctypes.addressof(U.desc), M, ctypes.addressof(x.desc), ctypes.addressof(y.desc), Coef(0.7, None),
           n, ctypes.addressof(v), ctypes.addressof(c), sums.data_ptr(), ndq.ndq._stream())
    assert rc == 0
    return sums


@pytest.mark.parametrize("block", [0, 64, 256])
@pytest.mark.parametrize("prec,lp,recon", [(ndq.F64, ndq.F64, 18), (ndq.F64, ndq.F64, 8), (ndq.F32, ndq.F32, 12),
                                           (ndq.F16, ndq.F16, 12), (ndq.F16, ndq.F32, 8)])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 10, 4, 6)])
@pytest.mark.parametrize("extra", [0, 1, 2, 3])
def test_sums_of_the_stored_field(dims, prec, lp, recon, block, extra):
    v = geometry.volume(dims)
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, torch.from_numpy(synthetic.gauge_field(dims, seed=111)).cuda(), lp, recon)
    x, *w = [ndq.SpinorField.pack(g, torch.from_numpy(synthetic.spinor(v, seed=112 + k)).cuda(), prec, ndq.FULL)
             for k in range(extra + 1)]
    y = w[-1] if extra > 1 else x.like()   # the last vector may be the output itself
    per = 64 if block == 0 else block
    blocks = 2 * -(-(v // 2) // per)
    ndq.set_launch(block, True)
    try:
        sums = q_combo(g, U, x, y, w).cpu().numpy()
    finally:
        ndq.set_launch(0, True)
    out = y.unpack().cpu().numpy()
    norm = (out.real ** 2 + out.imag ** 2).sum()
    assert np.isnan(sums[blocks:]).all()
    assert abs(sums[:blocks].sum() - norm) <= 1e-13 * norm
