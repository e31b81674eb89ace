"""The conversions on the matrix cores: the byte form of sources and constants and the reduction of its sums replayed with Python
integers at the largest moduli, and GPU parity where the kernel's pairs of targets, groups of sources and reductions have edges."""
import random

import pytest

import test_gpu_two_pass_rings as calls

gpu_only = pytest.mark.gpu


def _bytes(v, n=8):
    """v as n bytes in [-128, 127], least significant first."""
    out = []
    for _ in range(n):
        b = (v + 128) % 256 - 128
        out.append(b)
        v = (v - b) >> 8
    assert v == 0
    return out


def _centred(v, m):
    v %= m
    return v - m if v > m // 2 else v


def _sums(ys, cs, m, nbytes):
    """The eight 32-bit sums of a target: bytes of the sources times bytes of C_ki = c_k 2^(8 i) mod m."""
    s = [0] * 8
    for y, c in zip(ys, cs):
        for i, b in enumerate(_bytes(y, nbytes)):
            for p, e in enumerate(_bytes(_centred(c << (8 * i), m))):
                s[p] += b * e
    assert all(abs(v) <= 1 << 20 for v in s)
    return s


def _wrap(v, bits):
    return (v + (1 << (bits - 1))) % (1 << bits) - (1 << (bits - 1))


def _worst(rng, m, n):
    h = m // 2
    return [rng.choice((h, -h, h - rng.randrange(h), -rng.randrange(h))) for _ in range(n)]


@pytest.mark.parametrize("src_bits,bits", [(50, 60), (60, 60), (60, 51), (50, 52), (49, 36), (60, 37)])
def test_sums_to_an_integer_target(src_bits, bits):
    rng = random.Random(src_bits * 64 + bits)
    for m in ((1 << bits) - 1 - 2 * rng.randrange(1 << 20), (1 << (bits - 1)) + 1 + 2 * rng.randrange(1 << 20)):
        e = m.bit_length()
        sh = max(0, e - 51)
        mu = -(((1 << (64 + sh)) + m // 2) // m)
        for _ in range(60):
            cs = [rng.randrange(m) for _ in range(8)]
            ys = _worst(rng, (1 << src_bits) - 1, 8)
            s = _sums(ys, cs, m, 8)
            a = [s[2 * k] + (s[2 * k + 1] << 8) for k in range(4)]
            assert all(abs(v) < 1 << 31 for v in a)
            lo, hi = a[0] + (a[1] << 16), a[2] + (a[3] << 16)
            hi += lo >> 32
            lo &= 0xFFFFFFFF
            v = lo + (hi << 32)
            assert (v - sum(y * c for y, c in zip(ys, cs))) % m == 0 and abs(v) < m << 12
            t = hi >> sh
            assert -(1 << 31) <= t < 1 << 31 and -(1 << 31) <= mu < 0
            f = ((t * mu) >> 32) + 2
            x = (v + f * m) % (1 << 64)
            assert x == v + f * m and 0 <= x < 2.34 * m


@pytest.mark.parametrize("src_bits,bits", [(50, 50), (60, 50), (60, 30), (40, 20), (50, 40)])
def test_sums_to_a_double_precision_target(src_bits, bits):
    rng = random.Random(src_bits * 64 + bits)
    q = (1 << bits) - 1 - 2 * rng.randrange(1 << 10)
    qinv = 1.0 / q
    for _ in range(100):
        cs = [rng.randrange(q) for _ in range(8)]
        ys = _worst(rng, (1 << src_bits) - 1, 8)
        s = _sums(ys, cs, q, 7 if src_bits < 51 else 8)
        a = [s[2 * k] + (s[2 * k + 1] << 8) for k in range(4)]
        lo = a[0] + (a[1] << 16)
        hi = _wrap((lo >> 32) + a[2] + (a[3] << 16), 32)   # 32-bit words
        lo &= 0xFFFFFFFF
        v = lo + (hi << 32)
        assert (v - sum(y * c for y, c in zip(ys, cs))) % q == 0
        c = round(float(lo) * qinv + float(hi) * (qinv * 4294967296.0))
        d = (hi << 32) - c * q
        assert abs(d) <= 1 << 53
        x = d + lo
        assert (x - v) % q == 0 and abs(x) <= q / 2 + q * 2.0 ** -30


def test_bytes_of_double_precision_sources():
    """1.5 * 2^52 + v + 0x808080808080 holds six bytes plus 128 each and the seventh above them, for |v| < 2^49."""
    rng = random.Random(5)
    for v in [0, 1, -1, (1 << 49) - 1, 1 - (1 << 49)] + [rng.randrange(-(1 << 49), 1 << 49) for _ in range(200)]:
        t = (3 << 51) + v + 0x808080808080
        assert (1 << 52) <= t < 1 << 53
        word = (0x433 << 52) + t - (1 << 52)   # the bits of the double
        lo, hi = word & 0xFFFFFFFF ^ 0x80808080, ((word >> 32) ^ 0x8080) - 0x43380000 & 0xFFFFFFFF
        got = [(lo >> s) & 255 for s in (0, 8, 16, 24)] + [(hi >> s) & 255 for s in (0, 8, 16)]
        assert [b - 256 if b > 127 else b for b in got] == _bytes(v, 7)


SHAPES = [
    # (logN nq qbits np pbits dnum), nlimbs, B
    ((13, 5, 50, 5, 60, 1), 5, 1),     # two groups of sources, the second nearly empty; lone targets in every share
    ((13, 7, 50, 7, 60, 1), 7, 2),
    ((16, 6, 50, 5, 60, 1), 6, 1),     # the inverse pass apart
    ((14, 8, 60, 8, 50, 1), 8, 3),     # integer sources, double-precision targets, every group full
    ((13, 8, 30, 3, 60, 1), 8, 2),     # 30-bit primes
    ((15, 3, 52, 1, 52, 3), 3, 5),     # one source, 52-bit integers
    ((13, 9, 40, 3, 50, 3), 7, 30),    # a short last digit, one share of an odd number of targets
]


@gpu_only
@pytest.mark.parametrize("shape,nl,B", SHAPES)
def test_calls_around_the_products(shape, nl, B):
    calls.test_calls_on_the_smaller_two_pass_rings(shape, nl, B)
