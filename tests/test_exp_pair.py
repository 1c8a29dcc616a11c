"""The plain path's exponential, its steps in float32 as the kernels take them, against e^p in
float64 (CPU): within 1.5 units in the last place wherever the result is a normal number (the
hardware's 2^x stands in as correctly rounded; half a unit is its own rounding, the rest the
argument's), never at or above 1/255 of an opacity below the clamp, and NaN for NaN."""
import numpy as np
import pytest

f32 = np.float32
HI = f32(1.4426950408889634)
LO = f32(1.4426950408889634074 - float(HI))


def fma(a, b, c):
    return (a.astype(np.float64) * np.float64(b) + c.astype(np.float64)).astype(f32)


def exp_pair(p):
    q = np.where(p < f32(-200.0), f32(-200.0), p)
    hi = q * HI
    lo = fma(q, LO, fma(q, HI, -hi))
    n = np.rint(hi)
    with np.errstate(invalid="ignore", under="ignore"):
        e = np.exp2(((hi - n) + lo).astype(np.float64)).astype(f32)
        return np.ldexp(e, np.nan_to_num(n).astype(np.int32))


@pytest.mark.parametrize("lo,hi", [(-1e-6, 0.0), (-1.0, 0.0), (-6.0, -1.0), (-87.0, -6.0)])
def test_within_an_ulp(lo, hi):
    p = np.random.default_rng(1).uniform(lo, hi, 200_000).astype(f32)
    want = np.exp(p.astype(np.float64))
    err = np.abs(exp_pair(p).astype(np.float64) - want) / np.spacing(want.astype(f32)).astype(np.float64)
    assert err.max() <= 1.5


def test_far_below_and_not_a_number():
    p = np.array([-87.5, -104.0, -200.0, -201.0, -1e5, -1e9, -3e9, -1e12, -3e38, -np.inf], f32)
    assert np.all(exp_pair(p) < 1e-37)
    assert np.isnan(exp_pair(np.array([np.nan], f32)))[0]
