"""Gram matrices at the block sizes where the kernel changes its shape (elements
per stage, column tiles, wavefronts that share a row tile) and on lattices whose
sites are not whole stages or fewer than the wavefronts of a workgroup, against
numpy's products.  Tolerance: 12 V products of size about 1 summed in FP64 in
any order, 1e-13 of |A_i| |B_j| = 12 V."""
import numpy as np
import pytest

import synthetic
from oracle import geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 10, 2), (4, 6, 6, 10)])
@pytest.mark.parametrize("na,nb", [(16, 17), (17, 16), (20, 12), (9, 30), (32, 32), (33, 2), (40, 17), (48, 48), (33, 64),
                                   (3, 60)])
def test_gram_shapes(dims, na, nb):
    v = geometry.volume(dims)
    a = synthetic.spinor(v, nrhs=na, seed=91)
    b = synthetic.spinor(v, nrhs=nb, seed=92)
    g = ndq.Geometry(dims)
    A = ndq.SpinorField.pack(g, torch.from_numpy(a).cuda(), ndq.F64, ndq.FULL)
    B = ndq.SpinorField.pack(g, torch.from_numpy(b).cuda(), ndq.F64, ndq.FULL)
    G = ndq.spinor_gram(g, A, B).cpu().numpy()
    ref = a.reshape(na, -1).conj() @ b.reshape(nb, -1).T
    assert np.abs(G - ref).max() <= 1e-13 * 12 * v


@pytest.mark.parametrize("dims,na,nb", [((2, 2, 2, 2), 34, 3), ((6, 4, 10, 2), 48, 33), ((4, 6, 6, 10), 33, 20),
                                        ((8, 16, 16, 16), 41, 40), ((2, 2, 2, 2), 2, 4), ((4, 6, 6, 10), 4, 1),
                                        ((4, 6, 6, 10), 5, 8), ((8, 16, 16, 16), 3, 3), ((8, 16, 16, 16), 8, 2)])
def test_gram_three_row_tiles_and_small_blocks(dims, na, nb):
    v = geometry.volume(dims)
    rng = np.random.default_rng(93)
    a = rng.standard_normal((na, v, 4, 3)) + 1j * rng.standard_normal((na, v, 4, 3))
    b = rng.standard_normal((nb, v, 4, 3)) + 1j * rng.standard_normal((nb, v, 4, 3))
    g = ndq.Geometry(dims)
    A = ndq.SpinorField.pack(g, torch.from_numpy(a).cuda(), ndq.F64, ndq.FULL)
    B = ndq.SpinorField.pack(g, torch.from_numpy(b).cuda(), ndq.F64, ndq.FULL)
    G = ndq.spinor_gram(g, A, B).cpu().numpy()
    ref = a.reshape(na, -1).conj() @ b.reshape(nb, -1).T
    assert np.abs(G - ref).max() <= 1e-13 * 12 * v
