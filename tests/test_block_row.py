"""The block-row and workgroup divisions by multiplication (block_row, divide):
the same integer formulas over every value they are used for."""
import numpy as np


def test_block_row_is_the_quotient():
    t = np.arange(1024, dtype=np.uint64)
    for nx in range(1, 1025):
        inv = ((1 << 20) + nx - 1) // nx
        assert inv < 1 << 24 and int(t[-1]) * inv < 1 << 32     # a 24-bit product in 32 bits
        assert np.array_equal((t * np.uint64(inv)) >> np.uint64(20), t // np.uint64(nx)), nx


def test_divide_is_the_quotient():
    rng = np.random.default_rng(3)
    n = np.concatenate([rng.integers(0, 1 << 31, 4000), np.arange(300), (1 << 31) - 1 - np.arange(300)]).astype(np.uint64)
    for d in list(range(1, 400)) + [int(x) for x in rng.integers(400, 1 << 31, 400)] + [(1 << 31) - 1]:
        m = np.concatenate([n, np.uint64(d) * np.arange(1, 50, dtype=np.uint64) - np.uint64(1)])
        m = m[m < (1 << 31)]
        inv = 0xFFFFFFFF if d == 1 else (1 << 32) // d
        q = (m * np.uint64(inv)) >> np.uint64(32)
        r = m - q * np.uint64(d)
        short = r >= d
        q, r = q + short, r - short * np.uint64(d)
        assert np.array_equal(q, m // np.uint64(d)) and np.array_equal(r, m % np.uint64(d)), d
