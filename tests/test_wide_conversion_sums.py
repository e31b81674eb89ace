"""Conversions of more than 8 sources: joining and reducing the sums of bytes, replayed with Python integers at the most sources."""
import random
from fractions import Fraction

import pytest

from test_conversion_products import _bytes, _centred, _worst


def _sums(ys, cs, m):
    """The eight 32-bit sums of a target: bytes of the sources times bytes of C_ki = c_k 2^(8 i) mod m."""
    s = [0] * 8
    for y, c in zip(ys, cs):
        for i, b in enumerate(_bytes(y, 8)):
            for p, e in enumerate(_bytes(_centred(c << (8 * i), m))):
                s[p] += b * e
    assert all(abs(v) <= len(cs) << 17 for v in s)
    return s


def _turned(cs, m, p):
    """Sources of 8 bytes, below 2^59 in magnitude, whose products with byte p of their constants are all of one sign."""
    ys = []
    for c in cs:
        bs = [_bytes(_centred(c << (8 * i), m))[p] for i in range(8)]
        y = sum((127 if b > 0 else -128) << (8 * i) for i, b in enumerate(bs[:7]))
        ys.append(y + ((7 if bs[7] > 0 else -7) << 56))
    return ys


@pytest.mark.parametrize("n", [9, 45, 48])
@pytest.mark.parametrize("bits", [20, 40, 50, 51, 52, 60])
def test_sums_of_many_sources(n, bits):
    """More than 8 sources: sums of the pairs of bytes in 32-bit words, three words to a value, canonical residues of both kinds of
    targets. At 48 sources of the largest bytes a pair's sum is within int32 whatever the constants."""
    assert all(n * 8 * 128 * 128 * 257 < 1 << 31 for n in (45, 48))
    rng = random.Random(n * 64 + bits)
    for m in ((1 << bits) - 1 - 2 * rng.randrange(1 << 10), (1 << (bits - 1)) + 1 + 2 * rng.randrange(1 << 10)):
        for trial in range(14):
            cs = [rng.choice((m // 2, m // 2 + 1, rng.randrange(m))) if trial % 2 else rng.randrange(m) for _ in range(n)]
            if trial < 8:
                ys = _turned(cs, m, trial)
            elif trial < 11:   # the largest value: every product of the largest source with its constant's sign
                ys = [((1 << 59) - 1) * (1 if _centred(c, m) > 0 else -1) for c in cs]
            else:
                ys = _worst(rng, (1 << 60) - 1, n)
            if trial % 3 == 0:
                ys = [-y for y in ys]
            s = _sums(ys, cs, m)
            a = [s[2 * k] + (s[2 * k + 1] << 8) for k in range(4)]
            pair = a[0] + (a[1] << 16)
            lo, mid, top = pair & 0xFFFFFFFF, a[2] + (pair >> 32), a[3]
            assert all(-(1 << 31) <= v < 1 << 31 for v in a + [mid])
            v = lo + (mid << 32) + (top << 48)
            assert (v - sum(y * c for y, c in zip(ys, cs))) % m == 0
            if m >> 50 == 0:
                q, qinv, h = float(m), 1.0 / m, float(top * 65536 + mid)
                assert int(h) == top * 65536 + mid
                c = round(float(Fraction(lo) * Fraction(qinv) + Fraction(h * (qinv * 4294967296.0))))
                rest = Fraction(h) - c * Fraction(m, 1 << 32)
                assert Fraction(float(rest)) == rest
                x = rest * (1 << 32) + lo
                assert Fraction(float(x)) == x and -m < x < 2 * m
                x = int(x) + m if x < 0 else int(x)
                x = x - m if x >= m else x
            else:
                e = m.bit_length()
                sh = e - 48
                mu = -(((1 << (64 + sh)) + m // 2) // m)
                t = ((top << 16) + mid) >> sh
                assert -(1 << 31) <= t < 1 << 31 and -(1 << 31) <= mu < 0
                x = v + (((t * mu) >> 32) + 2) * m
                assert 0 <= x < 3 * m
                x = x - m if x >= m else x
                x = x - m if x >= m else x
            assert x == v % m
