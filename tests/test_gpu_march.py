"""The march along x0 of the multi-right-hand-side Q (work order 3) against the
one-lane-per-site kernel and the tile form: the same arithmetic in the same
order, so bit for bit.  The lattices have slices of less than a tile, of whole
tiles and of a ragged last one, the smallest x0 extent and several segments."""
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


@pytest.mark.parametrize("lp,recon", [(ndq.F32, 18), (ndq.F32, 12), (ndq.F32, 8), (ndq.F16, 18), (ndq.F16, 12)])
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 4, 6), 3), ((4, 2, 2, 2), 5), ((6, 4, 4, 8), 4), ((10, 6, 10, 6), 7),
                                       ((34, 4, 8, 4), 12)])
def test_march_equals_one_lane_kernel(dims, nrhs, lp, recon):
    v = geometry.volume(dims)
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, cu(synthetic.gauge_field(dims, seed=31)), lp, recon)
    psi = synthetic.spinor(v, nrhs=nrhs, seed=32)
    x = ndq.SpinorField.pack(g, cu(psi), ndq.F32, ndq.FULL)
    y = x.like()
    ndq.ndq.set_mrhs_launch(g, ndq.F32, lp, recon, nrhs, 2, 0, 3)
    ndq.apply_Q(g, U, M, x, y)
    rb = g.spinor_bytes(ndq.F32, ndq.FULL, 1)
    ndq.set_launch(64, 1)
    try:
        for r in range(nrhs):
            one = ndq.SpinorField.pack(g, cu(psi[r]), ndq.F32, ndq.FULL)
            out = one.like()
            ndq.apply_Q(g, U, M, one, out)
            assert torch.equal(y.buf[r * rb:(r + 1) * rb], out.buf), f"field {r}"
    finally:
        ndq.set_launch(0, 1)


@pytest.mark.parametrize("nrhs", [3, 60])
def test_march_many_slices_per_workgroup(nrhs):
    """60 fields fill the device with whole columns of 8 slices; 3 with shorter segments."""
    dims = (8, 16, 16, 16)
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, cu(synthetic.gauge_field(dims, seed=33)), ndq.F32, 12)
    x = ndq.SpinorField(g, ndq.F32, ndq.FULL, nrhs)
    gen = torch.Generator(device="cuda").manual_seed(34)
    x.buf.view(torch.float32).normal_(generator=gen)
    out = []
    for order in (3, 1):
        y = x.like()
        ndq.ndq.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2, 6, order)
        ndq.apply_Q(g, U, M, x, y)
        out.append(y.buf)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("recon", [18, 12])
@pytest.mark.parametrize("dims,nrhs", [((6, 4, 4, 8), 4), ((10, 6, 10, 6), 6)])
def test_march_with_extra_vectors(dims, nrhs, recon):
    """Clenshaw's recurrence fuses two and then three vectors into Q, the last of them the output itself."""
    v = geometry.volume(dims)
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, cu(synthetic.gauge_field(dims, seed=35)), ndq.F32, recon)
    x = ndq.SpinorField.pack(g, cu(synthetic.spinor(v, nrhs=nrhs, seed=36)), ndq.F32, ndq.FULL)
    ov = ndq.Overlap(g, M, ndq.Approx(ndq.MINMAX_POLY, 0.01, 7), 6.6)
    out = []
    for order in (3, 1):
        y = x.like()
        ndq.ndq.set_mrhs_launch(g, ndq.F32, ndq.F32, recon, nrhs, 2, 0, order)
        ndq.apply_sign(g, U, ov, x, y)
        out.append(y.buf)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("recon", [18, 12])
@pytest.mark.parametrize("dims,nrhs", [((6, 4, 4, 8), 8), ((10, 6, 10, 6), 11), ((2, 2, 4, 6), 9)])
def test_march_with_extra_vectors_in_several_groups(dims, nrhs, recon):
    """From 8 fields on launches with extra vectors march too; one field idle, none, and a group of three."""
    test_march_with_extra_vectors(dims, nrhs, recon)
