"""The quantizing kernels' way to the quotient of Eq. 1, in numpy: a reciprocal off by up to one ulp, a product and one
correction by the remainder must give the correctly rounded fp32 quotient for every difference of two fp16 values and every
fp16 scale that can meet."""
import numpy as np
import pytest

F = np.float32


def fma(a, b, c):
    """One rounding: the product of two fp32 numbers is exact in 64 significant bits, and so is the sum where the remainder
    is small against the product's terms."""
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(F)


@pytest.mark.parametrize("levels", [3, 15, 255, 65535, None])
@pytest.mark.parametrize("ulp", [-1, 0, 1])
def test_corrected_quotient_is_the_ieee_one(levels, ulp):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision here")
    rng = np.random.default_rng([levels or 0, ulp + 1])
    n = 1 << 18
    half = lambda: rng.integers(0, 0x7c00, n, dtype=np.uint16).view(np.float16).astype(F)
    hi, lo = half(), -half()
    if levels:  # the scale that belongs to a group from lo to hi, an element of the group
        S = ((hi - lo) / F(levels)).astype(np.float16).astype(F)
        x = np.clip((lo + (hi - lo) * rng.random(n).astype(F)), -65504, 65504).astype(np.float16).astype(F)
        d = np.maximum(x - lo, 0)
    else:       # any scale with any difference
        S, d = half(), hi - lo
    S = np.where(S == 0, F(2.0 ** -24), S)
    y = (1.0 / S.astype(np.float64)).astype(F)
    if ulp:
        y = np.nextafter(y, F(0) if ulp < 0 else F(np.inf))
    t = d * y
    q = fma(fma(-t, S, d), y, t)
    assert np.array_equal(q, (d.astype(np.float64) / S.astype(np.float64)).astype(F))  # 53 bits: rounds like fp32 division
