"""The default work order of the multi-right-hand-side stencil, asked of the library
without a launch: the march along x0 (order 3) gives a lane to every site of a slice
and rounds up to 64, so it is no default where the slices leave most lanes idle."""
import pytest

import paper_1010_5636_amd as ndq

THIN = [(4096, 2, 2, 2), (1024, 4, 2, 2), (512, 2, 2, 8), (256, 4, 4, 4), (1024, 4, 4, 4), (1024, 6, 6, 4),
        (800, 4, 4, 10), (2, 2, 2, 2)]


@pytest.mark.parametrize("dims", THIN)
def test_thin_slices_stay_tiles(dims):
    g = ndq.Geometry(dims)
    for recon in (18, 12, 8):
        for nrhs in list(range(2, 25)) + [32, 40, 60, 64, 1000]:
            got = ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, recon, nrhs, 2)
            assert got["group_major"] != 3, (dims, nrhs)


@pytest.mark.parametrize("dims,nrhs", [((64, 32, 32, 32), 12), ((48, 24, 24, 24), 12), ((48, 24, 24, 24), 4),
                                       ((32, 16, 16, 16), 12), ((32, 16, 16, 16), 8), ((10, 14, 20, 40), 9),
                                       ((600, 6, 6, 6), 24)])
def test_full_columns_march(dims, nrhs):
    g = ndq.Geometry(dims)
    assert ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2)["group_major"] == 3
    assert ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 1)["group_major"] != 3   # one output parity
    assert ndq.ndq.get_mrhs_launch(g, ndq.F64, ndq.F64, 12, nrhs, 2)["group_major"] != 3
    assert ndq.ndq.get_mrhs_launch(g, ndq.F16, ndq.F16, 12, nrhs, 2)["group_major"] != 3


@pytest.mark.parametrize("dims,nrhs", [((16, 14, 14, 14), 24), ((16, 12, 12, 12), 40), ((200, 6, 6, 10), 16),
                                       ((1024, 4, 4, 8), 6), ((32, 16, 16, 16), 7), ((48, 24, 24, 24), 5)])
def test_blocks_that_the_caches_hold_stay_tiles(dims, nrhs):
    g = ndq.Geometry(dims)
    assert ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 12, nrhs, 2)["group_major"] != 3
