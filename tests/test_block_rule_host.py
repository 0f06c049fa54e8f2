"""The rule that lets passes run as one block launch, on the host: which axes
of a default plan it covers, on both sides of each of its limits."""
import ctypes

import pytest

from paper_1501_07350_amd import _lib

C128, C64 = 0, 1
LDS = 160 * 1024   # bytes per workgroup on MI355X


def fused(A, B, C, grids, dtype):
    f = _lib.load().offt_test_fuse_rule
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 5
    f.restype = ctypes.c_int
    return f(dtype, A, B, C, grids, LDS)


def threads(A, B, C, blocks, dtype, streamed=0):
    f = _lib.load().offt_test_block_threads
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_int64]
    f.restype = ctypes.c_int
    return f(dtype, A, B, C, blocks, streamed, LDS)


@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_tiny_blocks(dtype):
    """Few tiny blocks gain a launch; many cost a workgroup each."""
    assert fused(2, 2, 2, 8192, dtype) == 3 and fused(2, 2, 2, 8193, dtype) == 0
    assert fused(1, 2, 2, 8192, dtype) == 2 and fused(1, 2, 2, 8193, dtype) == 0
    assert fused(512, 4, 4, 16, dtype) == 2 and fused(512, 4, 4, 17, dtype) == 0
    # 16^3 and 16 x 16 in any number
    assert fused(16, 16, 16, 1 << 16, dtype) == 3 and fused(1, 16, 16, 1 << 18, dtype) == 2


def test_blocks_between():
    # 144 points: 1152 bytes (up to 16384 of them in the caches), 2304 bytes
    assert fused(1, 12, 12, 16384, C64) == 2 and fused(1, 12, 12, 16385, C64) == 0
    assert fused(1, 12, 12, 16385, C128) == 2
    # streaming, 100 points are enough (300000 x 100 x 8 bytes < 256 MiB < 400000)
    assert fused(1, 20, 5, 300000, C64) == 0 and fused(1, 20, 5, 400000, C64) == 2
    assert fused(1, 18, 5, 600000, C64) == 0


@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_a_launch_holds_fewer_than_2_32_threads(dtype):
    """2^26 workgroups of 64 threads are refused by the runtime; the passes one
    by one need fewer."""
    for A, B, C, naxes in ((1, 16, 16, 2), (1, 16, 8, 2), (8, 8, 8, 3), (2, 2, 2, 3)):
        for grids in (1 << 20, 1 << 22, 1 << 25, (1 << 26) - 1, 1 << 26, 1 << 28):
            f = fused(A, B, C, grids, dtype)
            if f:
                assert f == naxes
                for s in (0, 1):
                    t = threads(A, B, C, grids, dtype, s)
                    assert t >= 64 and grids * t < 1 << 32
        assert fused(A, B, C, 1 << 26, dtype) == 0


def test_few_planes_that_fill_a_cu():
    # 128 x 128 complex64 fills a CU's LDS and its threads: from 80 planes to
    # 256, or streaming; 100 x 120 leaves threads idle: from 128
    assert fused(79, 128, 128, 1, C64) == 0 and fused(80, 128, 128, 1, C64) == 2
    assert fused(127, 100, 120, 1, C64) == 0 and fused(128, 100, 120, 1, C64) == 2
    assert fused(1, 128, 128, 257, C64) == 0 and fused(1, 128, 128, 4096, C64) == 2


def test_three_stage_lines_along_b():
    # 243 = 9 x 9 x 3: as the planes' columns up to 64 MiB, as rows always
    small, large = 64 * 2 ** 20 // (243 * 20 * 8), 64 * 2 ** 20 // (243 * 20 * 8) + 1
    assert fused(1, 243, 20, small, C64) == 2 and fused(1, 243, 20, large, C64) == 0
    assert fused(1, 20, 243, large, C64) == 2


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
