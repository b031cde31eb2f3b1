"""The grid corner from one reciprocal product (denominators 2 * blocks up to 2^18 that are no power of
two), as the kernels take it, against integer division and the correctly rounded quotient."""
import numpy as np
import pytest

F32 = np.float32


def corner_rcp(b, blocks, res):
    den = 2 * blocks
    num = (2 * b + 1) * res - blocks
    inv = F32(1.0) / F32(den)
    q = (num.astype(F32) * inv).astype(np.int64)  # truncation, as the kernel's conversion
    rem = num - q * den
    q, rem = np.where(rem < 0, q - 1, np.where(rem >= den, q + 1, q)), np.where(rem < 0, rem + den, np.where(rem >= den, rem - den, rem))
    a = rem.astype(F32)
    q0 = (a * inv).astype(F32)
    # the two fused steps in float64: the products of 24-bit values are exact there
    e = (a.astype(np.float64) - float(den) * q0.astype(np.float64)).astype(F32)
    f = (q0.astype(np.float64) + e.astype(np.float64) * float(inv)).astype(F32)
    return q, f


@pytest.mark.parametrize("blocks", [1, 3, 5, 7, 64, 125, 275, 333, 500, 1023, 1025, 4095, 12345, 65535, 131071])
@pytest.mark.parametrize("res", [2, 8, 13, 256, 2048, 8191])
def test_corner_by_reciprocal(blocks, res):
    if (2 * blocks + 1) * res >= 1 << 31:
        pytest.skip("taken by the 64-bit path")
    b = np.arange(blocks, dtype=np.int64)
    if blocks > 20000:
        b = np.unique(np.random.default_rng(blocks + res).choice(blocks, 20000))
    den = 2 * blocks
    num = (2 * b + 1) * res - blocks
    inside = (num > 0) & (num < (res - 1) * den)
    q, f = corner_rcp(b, blocks, res)
    want_q = num // den
    want_f = (num - want_q * den).astype(F32) / F32(den)
    assert np.array_equal(q[inside], want_q[inside])
    assert np.array_equal(f[inside], want_f[inside])
