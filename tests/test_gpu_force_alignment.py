"""The link force goes into any array of doubles, one that starts between two
16-byte words too; and nothing around it is written."""
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


@pytest.mark.parametrize("with_grad", [False, True])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 6, 2, 10), (6, 4, 4, 6)])
def test_force_between_two_words(dims, with_grad):
    nb = ndq.ndq
    v = geometry.volume(dims)
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, torch.from_numpy(synthetic.gauge_field(dims, seed=61)).cuda(), ndq.F64, 18)
    a, b = (ndq.SpinorField.pack(g, torch.from_numpy(synthetic.spinor(v, seed=s)).cuda(), ndq.F64, ndq.FULL)
            for s in (62, 63))
    ref, gref = ndq.gauge_force(g, U, a, b, want_force=True, want_grad=True)
    n = v * 4 * 8
    buf = torch.full((n + 4,), np.nan, dtype=torch.float64, device="cuda")
    for off in (1, 2, 3):
        buf.fill_(np.nan)
        out = buf[off:off + n]
        grad = torch.empty_like(gref) if with_grad else None
        rc = nb.lib().ndq_gauge_force(g.handle, ctypes.byref(U.desc), ctypes.byref(a.desc), ctypes.byref(b.desc),
                                      ctypes.c_void_p(out.data_ptr()),
                                      ctypes.c_void_p(grad.data_ptr()) if with_grad else None, nb._stream())
        assert rc == 0
        assert torch.equal(out, ref.reshape(-1))
        assert torch.isnan(buf[:off]).all() and torch.isnan(buf[off + n:]).all()
        if with_grad:
            assert torch.equal(grad, gref)
