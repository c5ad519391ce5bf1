"""Slices per workgroup of the march along x0: the host function against a search
through every number of slices, and its time where n0 is long (it runs on every
launch).  Called by its C++ name: it is no entry point of the library."""
import ctypes
import time

import pytest

import paper_1010_5636_amd as ndq


@pytest.fixture(scope="module")
def march_slices():
    f = getattr(ndq.ndq.lib(), "_ZN3ndq12march_slicesEili")   # ndq::march_slices(int, int64_t, int)
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    return f


def search(n0, columns, resident):
    """The smallest T with the fewest steps: rounds of resident workgroups times 2 T + 3."""
    return min(range(1, n0 + 1), key=lambda t: -(-columns * -(-n0 // t) // resident) * (2 * t + 3))


@pytest.mark.parametrize("resident", [1, 7, 512])
def test_equals_the_search_through_all(march_slices, resident):
    for n0 in (2, 4, 6, 10, 16, 22, 48, 64, 130, 254):
        for columns in (2, 4, 6, 14, 32, 88, 216, 510, 512, 514, 648, 1024, 1536, 6144, 12290):
            assert march_slices(n0, columns, resident) == search(n0, columns, resident), (n0, columns)


@pytest.mark.parametrize("columns", [2, 6, 30, 1000, 2502])
def test_long_lattices_take_no_host_time(march_slices, columns):
    """A loop through 2^20 numbers of slices took some milliseconds."""
    best = 1.0
    for _ in range(5):
        t0 = time.perf_counter()
        march_slices(1 << 20, columns, 512)
        best = min(best, time.perf_counter() - t0)
    assert best < 5e-4, best
