"""Host-side check of the weight-gradient workspace (no GPU): a trainer allocates it
once, for its largest batch, and every batch up to that one has to fit.

The number of partial matrices of a launch, n products times ceil(B / chunk length), is
not monotone in B, because the chunk length is rounded up to whole 64-sample tiles:
1,345 samples take 11 chunks where 1,344 take 21."""
import ctypes

import pytest

import paper_2601_18548_amd as g

WIDTH = 256


@pytest.fixture(scope="module")
def sizes():
    lib = g.library()
    chunk_len = lib._ZN4gcdf15wgrad_chunk_lenEliii
    chunk_len.restype, chunk_len.argtypes = ctypes.c_int64, [ctypes.c_int64] + [ctypes.c_int] * 3
    floats = lib._ZN4gcdf20wgrad_partial_floatsElii
    floats.restype, floats.argtypes = ctypes.c_int64, [ctypes.c_int64] + [ctypes.c_int] * 2
    return chunk_len, floats


@pytest.mark.parametrize("num_cu", [256, 64, 4, 1])
def test_every_smaller_batch_fits_the_workspace_of_the_largest(sizes, num_cu):
    chunk_len, floats = sizes
    most = 0  # matrices that some batch so far has needed
    for B in range(1, 26001):
        for n in (1, 2, 3):
            L = chunk_len(B, n, WIDTH, num_cu)
            assert L >= 64 and L % 64 == 0  # chunks start at whole tiles
            most = max(most, n * -(-B // L))
        assert floats(B, WIDTH, num_cu) >= most * WIDTH * WIDTH, "a trainer of max_batch %d is short" % B
