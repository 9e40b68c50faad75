"""The quantiser's quotient without a division, over every pair of fp16 mantissas."""
import numpy as np


def fma32(a, b, c):
    """a * b + c rounded once to float32, for float32 arrays whose products are exact in
    float64 (two 24-bit factors): the sum's float64 rounding error decides ties."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    r = s.astype(np.float32)
    back = r.astype(np.float64)
    other = np.nextafter(r, np.where(s > back, np.inf, -np.inf).astype(np.float32)).astype(np.float64)
    tie = (s != back) & (s - back == other - s)
    towards = tie & (err != 0) & (np.sign(err) == np.sign(other - back))
    return np.where(towards, other.astype(np.float32), np.where(tie & (err != 0) & ~towards, back.astype(np.float32), r))


def test_reciprocal_quotient_equals_the_division():
    """q0 = v r with r = 1 / s, then q0 + (v - q0 s) r, is the float32 quotient v / s for all
    1024 x 1024 mantissas (exponents only scale it: no product here is subnormal), and the
    sum with 1.5 * 2^23 holds its integer, ties to even, for quotients below 128."""
    m = (1 + np.arange(1024, dtype=np.float32) / 1024).astype(np.float32)
    v, s = m[:, None] * np.ones_like(m), np.ones_like(m)[:, None] * m
    r = np.float32(1) / s
    q0 = v * r
    q = fma32(fma32(-q0, s, v), r, q0)
    assert np.array_equal(q, v / s)
    for e in range(-3, 7):  # quotients of 2^-4 to 128
        x = np.ldexp(q, e)
        assert x.max() < 128
        for sign in (np.float32(1), np.float32(-1)):
            for bias in (np.float32(12582912), np.float32(12582920)):  # INT8; INT4, whose nibbles are code + 8
                code = (sign * x + bias).view(np.int32) - bias.view(np.int32)
                assert np.array_equal(code, np.rint(sign * x).astype(np.int32))
