"""The quantizers' quotient (one correction of x times the scale's reciprocal) decides every E4M3
rounding as the float32 quotient does.

A code depends on x / sigma only through its place among the format's rounding boundaries, the
5-bit significands M (midpoints of neighbouring codes; the powers of two among them are midpoints
of subnormal codes), on either side or equal.  x has 8 significand bits and sigma 24.  The
corrected quotient is within a unit of the exact one, so only sigmas within a few units of x / M
can decide otherwise: all of those are enumerated, in exact arithmetic with every operation
rounded once to 24 bits (scaling by powers of two changes nothing: no operation underflows where
the code is not 0).
"""

from fractions import Fraction

import numpy as np


def rn24(v):
    """v > 0 or < 0 or 0 rounded to 24 significand bits, ties to even."""
    if v == 0:
        return v
    s = -1 if v < 0 else 1
    n, d = abs(v).numerator, abs(v).denominator
    e = n.bit_length() - d.bit_length() - 24
    q = Fraction(n, d) / Fraction(2) ** e
    if q >= 1 << 24:
        e += 1
        q /= 2
    k, rest = divmod(q.numerator, q.denominator)
    twice = 2 * rest
    if twice > q.denominator or (twice == q.denominator and k & 1):
        k += 1
    return s * k * Fraction(2) ** e


def corrected(x, sigma, y):
    q = rn24(x * y)
    rem = rn24(q * sigma - x)
    return rn24(q - rem * y)


def test_every_rounding_boundary():
    checked = 0
    for a in range(128, 256):
        for m in range(16, 32):
            at = Fraction(a, m)
            e = 0
            while at < 1 << 23:
                at *= 2
                e += 1
            assert at < 1 << 24
            for b in range(int(at) - 4, int(at) + 6):
                if not (1 << 23) <= b < (1 << 24):
                    continue
                sigma = Fraction(b)
                x = Fraction(a) * 2 ** e            # x / sigma is next to m
                want = rn24(x / sigma)
                got = corrected(x, sigma, rn24(1 / sigma))
                assert (got > m) - (got < m) == (want > m) - (want < m), (a, m, b)
                checked += 1
    assert checked > 15000


def test_within_a_unit_elsewhere():
    rng = np.random.default_rng(3)
    for _ in range(4000):
        x, sigma = Fraction(int(rng.integers(128, 256))), Fraction(int(rng.integers(1 << 23, 1 << 24)))
        want = rn24(x / sigma)
        got = corrected(x, sigma, rn24(1 / sigma))
        assert abs(got - want) <= want * Fraction(1, 1 << 23)
