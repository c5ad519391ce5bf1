"""The default tile order of the one-field kernels, asked of the library without a
launch and by its C++ name (it is no entry point): a dslash that the caches hold
runs in index order (16^3x32 is slower in the slice-chunked order in every format)."""
import ctypes

import pytest

import paper_1010_5636_amd as ndq

Q, DSLASH = 2, 1   # output parities


def order(dims, prec, parities):
    f = getattr(ndq.ndq.lib(), "_ZN3ndq13default_orderERKNS_5GeomKEii")   # default_order(const GeomK&, int, int)
    f.restype = ctypes.c_int
    n0, n1, n2, n3 = dims
    s1, s0 = n2 * n3 // 2, n1 * n2 * n3 // 2
    lattice = (ctypes.c_int32 * 64)(n0, n1, n2, n3, n3 // 2, s1, s0, n0 * s0)
    return f(lattice, ctypes.c_int(prec), ctypes.c_int(parities))


@pytest.mark.parametrize("prec", [ndq.F64, ndq.F32, ndq.F16])
def test_dslash_in_the_caches(prec):
    for dims in ((32, 16, 16, 16), (64, 16, 16, 8), (16, 16, 16, 16), (4, 4, 4, 4)):
        assert order(dims, prec, DSLASH) == 0, dims
        assert order(dims, prec, Q) == 1, dims


@pytest.mark.parametrize("prec", [ndq.F64, ndq.F32, ndq.F16])
def test_dslash_beyond_them(prec):
    assert order((48, 24, 24, 24), prec, DSLASH) == 1
    assert order((64, 48, 48, 48), prec, DSLASH) == 0   # three slices beyond an L2
