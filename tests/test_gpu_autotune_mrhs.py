"""The work-order autotuner of the multi-right-hand-side stencil tries every order
that a default may be: from any order in use it can come back to the default's."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402

DIMS = (8, 8, 8, 16)   # 8 tiles a slice: the two-row chunk is 2, so 3 chunks are tried


@pytest.fixture(scope="module")
def lattice():
    g = ndq.Geometry(DIMS)
    u = torch.from_numpy(np.ascontiguousarray(synthetic.gauge_field(DIMS))).cuda()
    return g, {p: ndq.GaugeField.pack(g, u, p, 12) for p in (ndq.F32, ndq.F64)}


@pytest.mark.parametrize("nrhs", [8, 20])
@pytest.mark.parametrize("prec,ny", [(ndq.F32, 2), (ndq.F32, 1), (ndq.F64, 2)])
def test_candidates(lattice, prec, ny, nrhs):
    g, U = lattice
    nb = ndq.ndq
    dflt = nb.get_mrhs_launch(g, prec, prec, 12, nrhs, ny)
    nb.set_mrhs_launch(g, prec, prec, 12, nrhs, ny, 1, 0, 0)   # one field per workgroup
    try:
        r = nb.autotune_mrhs(g, U[prec], prec, nrhs, ny, reps=3)
        groups = {k for k in (nrhs, (nrhs + 1) // 2, (nrhs + 2) // 3, 8, 6, 4, 2) if k <= nrhs}
        march = prec == ndq.F32 and ny == 2
        assert r["nshapes"] == sum(3 if k == nrhs else 6 for k in groups) + march
        assert r["us_best"] <= r["us_previous"]
    finally:
        nb.set_mrhs_launch(g, prec, prec, 12, nrhs, ny, **dflt)


def test_march_is_found_again():
    """16 fields on 16^3x32: 106 us marching, 147 in the fastest tile order."""
    dims, nrhs = (32, 16, 16, 16), 16
    g = ndq.Geometry(dims)
    nb = ndq.ndq
    U = ndq.GaugeField.pack(g, torch.from_numpy(synthetic.gauge_field(dims)).cuda(), ndq.F32, 12)
    dflt = nb.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2)
    assert dflt["group_major"] == 3
    nb.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2, 1, 0, 0)
    try:
        nb.autotune_mrhs(g, U, ndq.F32, nrhs, 2, reps=10)
        assert nb.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2)["group_major"] == 3
    finally:
        nb.set_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2, **dflt)
