"""The direction split on F16 storage: three wavefronts store a plane each under the
scale that the largest real of all three sets.  Point sources put that real into
each plane and leave sites without any; against the FP64 oracle within the storage's
rounding of the site's largest real, and exactly zero where Q reaches nothing."""
import numpy as np
import pytest

import synthetic
from oracle import dirac, geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402

M = -1.4


def cu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("recon", [18, 12])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 10, 4, 6)])
@pytest.mark.parametrize("comp", [0, 3, 4, 7, 8, 11])
def test_point_sources(dims, comp, recon):
    """Storing rounds to 2^-11 of the largest real of a site, the links to 2^-11 of theirs."""
    v = geometry.volume(dims)
    u = synthetic.gauge_field(dims, seed=41)
    psi = np.zeros((v, 4, 3), dtype=np.complex128)
    psi[v // 3, comp // 3, comp % 3] = 3.0
    g = ndq.Geometry(dims)
    U = ndq.GaugeField.pack(g, cu(u), ndq.F16, recon)
    x = ndq.SpinorField.pack(g, cu(psi), ndq.F16, ndq.FULL)
    y = x.like()
    ndq.apply_Q(g, U, M, x, y)
    got = y.unpack().cpu().numpy().reshape(v, 12)
    ref = dirac.apply_Q(u, psi, M, dims).reshape(v, 12)
    top = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=1)
    assert (got[top == 0] == 0).all()
    assert (np.abs(got - ref).max(axis=1) <= 5e-3 * 3.0).all()
    assert (top > 0).sum() > 1
