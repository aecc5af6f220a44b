"""Host check (no GPU): the launch and the workspace of the fill contraction.  Its blocks and partials are no
more than one per 64 x 64 entries of the product, the launch stays below 2^32 threads for every timeslice
that the entry points accept, and the waves' strided walk meets every 16 x 16 tile once."""
import ctypes
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1405_4524_amd", "_build", "liba2a.so")
MAX_ROWS = 1 << 21  # 12 X Y Z of the largest timeslice that the contraction accepts
STORE_MAX_ROWS = (1 << 18) - 1


@pytest.fixture(scope="module")
def blocks():
    if not os.path.exists(LIB):
        pytest.skip("the built library is missing")
    f = ctypes.CDLL(LIB)["_ZN3a2a11fill_blocksEii"]  # a2a::fill_blocks(int, int)
    f.restype = ctypes.c_int
    return lambda m: f(m, m)


def rows():
    """Rows of timeslices: 12 times products of three even extents, small, ordinary and the largest."""
    ext = [2, 4, 6, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 54, 56]
    return sorted({12 * x * y * z for x in ext for y in ext for z in ext if 12 * x * y * z <= MAX_ROWS})


def test_workspace_and_launch(blocks):
    for m in rows():
        n = blocks(m)
        assert 1 <= n <= ((m + 63) // 64) ** 2, m
        assert n * 256 < 1 << 32, m
    assert (STORE_MAX_ROWS // 96 * 96 // 32) ** 2 * 64 < 1 << 32


@pytest.mark.parametrize("m", [96, 192, 288, 768, 1152, 6144, 49152])
def test_every_tile_once(blocks, m):
    t, stride = m // 16, 4 * blocks(m)
    seen = np.zeros((t, t), np.int32)
    start = np.arange(stride)
    row, col = start // t, start % t
    while True:
        on = row < t
        if not on.any():
            break
        np.add.at(seen, (row[on], col[on]), 1)
        row, col = row + stride // t, col + stride % t
        over = col >= t
        row, col = row + over, col - over * t
    assert (seen == 1).all()
