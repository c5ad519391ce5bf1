"""Links that a multi-right-hand-side tile decodes once and stages in LDS: one
launch over several lattices against the one-lane-per-site kernel, which decodes
them in registers, so bit for bit."""
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


@pytest.mark.parametrize("prec", [ndq.F64, ndq.F32])
def test_eight_real_links_over_several_lattices(prec):
    jobs = []
    for k, (dims, nrhs) in enumerate([((2, 2, 2, 2), 2), ((4, 4, 4, 4), 1), ((6, 10, 4, 6), 5)]):
        g = ndq.Geometry(dims)
        U = ndq.GaugeField.pack(g, cu(synthetic.gauge_field(dims, seed=71 + k)), prec, 8)
        psi = synthetic.spinor(geometry.volume(dims), nrhs=nrhs, seed=81 + k)
        x = ndq.SpinorField.pack(g, cu(psi), prec, ndq.FULL)
        jobs.append((g, U, M, x, x.like(), psi))
    ndq.apply_Q_multi([j[:5] for j in jobs])
    ndq.set_launch(64, 1)
    try:
        for g, U, m, x, y, psi in jobs:
            rb = g.spinor_bytes(prec, ndq.FULL, 1)
            for r in range(psi.shape[0]):
                one = ndq.SpinorField.pack(g, cu(psi[r]), prec, ndq.FULL)
                out = one.like()
                ndq.apply_Q(g, U, m, one, out)
                assert torch.equal(y.buf[r * rb:(r + 1) * rb], out.buf), f"field {r}"
    finally:
        ndq.set_launch(0, 1)
