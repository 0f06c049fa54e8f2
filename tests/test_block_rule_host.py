"""Threads of a block launch, on the host."""
import ctypes

import pytest

from paper_1501_07350_amd import _lib

C128, C64 = 0, 1
LDS = 160 * 1024   # bytes per workgroup on MI355X


def threads(A, B, C, blocks, dtype, streamed=0):
    f = _lib.load().offt_test_block_threads
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_int64]
    f.restype = ctypes.c_int
    return f(dtype, A, B, C, blocks, streamed, LDS)


@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_threads(dtype):
    """Up to a block per CU a thread per line of the longest pass; beyond, not
    so many that a second workgroup does not fit."""
    most, B = (1024, 50) if dtype == C64 else (512, 25)
    assert threads(1, B, 125, 256, dtype) == most
    assert threads(1, B, 125, 4096, dtype) == most // 2
    for B, C in ((2, 2), (250, 2), (2, 250), (243, 20), (16, 16), (100, 32)):
        for blocks in (1, 256, 257, 1000, 100000):
            for s in (0, 1):
                t = threads(1, B, C, blocks, dtype, s)
                assert t % 64 == 0 and 64 <= t <= 1024
