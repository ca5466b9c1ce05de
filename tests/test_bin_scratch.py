"""The depth sort's digit counts lie in the part of the binning scratch that holds the
footprint ellipses afterwards (32 bytes a pair): their size is what the kernels index, and
fits."""
import ctypes

import pytest

from paper_2411_09156_amd import _lib


def _words(n, views):
    fn = ctypes.CDLL(_lib.LIB_PATH)["_ZN4gesr21depth_sort_hist_wordsEjj"]
    fn.restype, fn.argtypes = ctypes.c_uint64, [ctypes.c_uint32, ctypes.c_uint32]
    return fn(n, views)


@pytest.mark.parametrize("views", [1, 3, 32])
@pytest.mark.parametrize("n,keys", [(1, 0), (4096, 0), (4097, 1024), (65_536, 1024), (65_537, 2048), (131_072, 2048),
                                    (131_073, 4096), (262_145, 4096), (3_000_000, 4096)])
def test_digit_counts_fit_the_ellipses(n, keys, views):
    # a row of 256 counts per block of `keys` keys; none where a view is sorted in LDS
    blocks = -(-n // keys) if keys else 0
    assert _words(n, views) == views * blocks * 256 <= 8 * n * views
