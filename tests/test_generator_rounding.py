"""The square root and the division of the normal transform (csrc/rng.hip: sqrt_unscaled, divide_unscaled) start from an
instruction that is accurate to 1 ulp and have to end at the correctly rounded value, which is what the CPU definition of the
generators computes.  Here both sequences run operation by operation on every argument that matters and from every estimate
such an instruction may return; numpy's float32 square root and division are correctly rounded.

A fused operation rounds once.  Its product of two float32 values is exact in float64; where the sum is not, the float64 result
is rounded to odd before it is rounded to float32 (53 >= 24 + 2 bits, so that no double rounding is left)."""
import numpy as np
import pytest

f32, f64 = np.float32, np.float64


def ulps(x, n):
    return (x.view(np.int32) + np.int32(n)).view(f32)


def fma(a, b, c):
    p, c = f64(a) * f64(b), f64(c)
    s = p + c
    t = s - p                                    # two-sum: s + err is the exact sum
    err = (p - (s - t)) + (c - t)
    bits = s.view(np.int64)
    even, away = (err != 0) & (bits & 1 == 0), (err > 0) == (s > 0)
    return (bits + np.where(even, np.where(away, 1, -1), 0)).view(f64).astype(f32)


@pytest.mark.parametrize("off", [-1, 0, 1])
@pytest.mark.parametrize("exponent", [0, 1])
def test_square_root_of_every_significand(exponent, off):
    x = ((np.arange(1 << 23, dtype=np.int32)) | np.int32((127 + exponent) << 23)).view(f32)
    ref = np.sqrt(x)
    r = ulps(ref, off)
    lo, hi = ulps(r, -1), ulps(r, 1)
    out = np.where(fma(-lo, r, x) <= 0, lo, r)
    out = np.where(fma(-hi, r, x) > 0, hi, out)
    assert np.array_equal(out, ref)


@pytest.mark.parametrize("off", [-1, 0, 1])
def test_division_of_every_significand(off):
    j = np.arange(1 << 23, 1 << 24, dtype=np.int32).astype(f32)
    bits = j.view(np.uint32) + np.uint32(0x3F800000 - 0x3F3504F4)
    m = ((bits & np.uint32(0x007FFFFF)) + np.uint32(0x3F3504F4)).view(f32)
    a, d = m - f32(1), m + f32(1)
    assert d.min() > 1.7 and d.max() < 2.5
    y = ulps(f32(1) / d, off)
    y = fma(fma(-d, y, f32(1)), y, y)
    q = a * y
    out = fma(fma(-d, q, a), y, q)
    # The largest d below 2, all ones, is the exception that Markstein's theorem has: its reciprocal has to be right to begin
    # with.  tests/test_gpu_generators.py draws it on the device.
    assert np.all((out == a / d) | ((d == ulps(f32([2]), -1)) & (off != 0)))
