"""The march along x0 where no other test takes it: launches with two and three extra
vectors on 8-real and F16 links, and the default route of a block that marches.  Bit
for bit against the tile form."""
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


def cu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("lp,recon", [(ndq.F32, 8), (ndq.F16, 18), (ndq.F16, 12)])
@pytest.mark.parametrize("dims,nrhs", [((6, 4, 4, 8), 8), ((10, 6, 10, 6), 11), ((2, 2, 4, 6), 9)])
def test_extra_vectors_in_other_link_formats(dims, nrhs, lp, recon):
    nb = ndq.ndq
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, cu(synthetic.gauge_field(dims, seed=121)), lp, recon)
    x = ndq.SpinorField.pack(g, cu(synthetic.spinor(geometry.volume(dims), nrhs=nrhs, seed=122)), ndq.F32, ndq.FULL)
    ov = ndq.Overlap(g, M, ndq.Approx(ndq.MINMAX_POLY, 0.01, 7), 6.6)
    dflt = nb.get_mrhs_launch(g, ndq.F32, lp, recon, nrhs, 2)
    out = []
    try:
        for order in (3, 1):
            nb.set_mrhs_launch(g, ndq.F32, lp, recon, nrhs, 2, 0, order)
            y = x.like()
            ndq.apply_sign(g, U, ov, x, y)
            out.append(y.buf)
    finally:
        nb.set_mrhs_launch(g, ndq.F32, lp, recon, nrhs, 2, **dflt)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dims,nrhs", [((20, 18, 18, 18), 9), ((32, 16, 16, 16), 8), ((10, 14, 20, 40), 13)])
def test_default_route(dims, nrhs):
    """Random reals for links: only the sums are compared."""
    nb = ndq.ndq
    g = ndq.Geometry(dims)
    gen = torch.Generator(device="cuda").manual_seed(123)
    U = ndq.GaugeField(g, ndq.F32, 12)
    U.buf.view(torch.float32).normal_(generator=gen)
    x = ndq.SpinorField(g, ndq.F32, ndq.FULL, nrhs)
    x.buf.view(torch.float32).normal_(generator=gen)
    dflt = nb.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2)
    assert dflt["group_major"] == 3
    ov = ndq.Overlap(g, M, ndq.Approx(ndq.MINMAX_POLY, 0.01, 3), 6.6)
    out = []
    try:
        for shape in (dflt, dict(dflt, group_major=1)):
            nb.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2, **shape)
            y, s = x.like(), x.like()
            ndq.apply_Q(g, U, M, x, y)
            ndq.apply_sign(g, U, ov, x, s)
            out.append((y.buf, s.buf))
    finally:
        nb.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2, **dflt)
    assert torch.isfinite(out[0][1].view(torch.float32)).all()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])
