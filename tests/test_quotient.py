"""The quantizer's division by the row's reciprocal (TokenQuantizer::quotient), step by step in binary32 on the host: the correctly
rounded quotient for every binary16 value over the steps that rows can have."""
import numpy as np
import pytest

f32, f64 = np.float32, np.float64


def fma(a, b, c):
    """binary32 fused multiply-add: the product of two binary32 is exact in binary64; the sum there is rounded to odd, so that the
    rounding to binary32 that follows is the only one."""
    p, c = a.astype(f64) * b.astype(f64), c.astype(f64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)                                 # (exactly what the sum left out)
    away = np.nextafter(s, np.where(err > 0, np.inf, -np.inf))
    even = (s.view(np.int64) & 1) == 0
    return np.where((err != 0) & even, away, s).astype(f32)


def quotient(x, delta, inv):
    t = x * inv
    t = fma(fma(-t, delta, x), inv, t)
    return fma(fma(-t, delta, x), inv, t)


def test_fma_rounds_once():
    one, e = np.array([f32(1)]), np.array([f32(2.0 ** -24)])
    up = np.array([np.nextafter(f32(1), f32(2))])
    assert fma(one, one, e)[0] == f32(1) and fma(up, one, e)[0] > up[0]              # ties to even
    assert fma(up, up, -(up * up))[0] == f32(2.0 ** -46)                             # the product's own rounding error


@pytest.mark.parametrize("q", [1, 2, 5, 8])
def test_quotient_is_correctly_rounded(q):
    """All halves of one sign (the steps are odd in x), the smallest and largest of a few hundred ranges among them."""
    rng = np.random.default_rng(q)
    halves = np.arange(1, 0x7C00, dtype=np.uint16).view(np.float16).astype(f32)
    tops = np.concatenate([halves[[0, 1, 2, 1022, 1023, 1024, -2, -1]], halves[rng.integers(0, halves.size, 160)]])
    lows = np.concatenate([np.zeros(8, f32), halves[-1:], halves[rng.integers(0, halves.size, 159)]])
    for lo, hi in zip(lows, tops):
        delta = (hi + lo) / f32((1 << q) - 1)                     # one sign's halves against either end of the range
        x = halves[halves <= max(lo, hi)]
        d = np.broadcast_to(delta, x.shape)
        inv = np.broadcast_to(f32(1) / delta, x.shape)
        assert delta > 0 and np.isfinite(inv).all()
        got, want = quotient(x, d, inv), x / d
        assert np.array_equal(got, want), (q, lo, hi, x[got != want][:3])
