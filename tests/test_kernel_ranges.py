"""Range arguments of the integer butterflies, replayed with Python integers (no GPU).

The HIP kernels keep lazy values in 64-bit words: the twiddle product estimates its quotient from three of the four
32 x 32 partial products (result below 4q), 60-bit primes use Harvey-style butterflies on [0,16q) / [0,8q), primes below
2^52 never correct on the way forward and let sums double on the way back. These tests follow the same recurrences at
the largest moduli each form accepts and check that nothing reaches 2^64 and that every value stays congruent to the
exact product. They model the arithmetic statement, not the kernels' code: bit-exactness of the kernels themselves is
what the GPU parity tests check.
"""
import random
from fractions import Fraction

M64 = (1 << 64) - 1


def approx_product(x, w, ws, m):
    """x * w - qt * m modulo 2^64, qt = top partial product + high words of the two middle ones of x * ws."""
    x0, x1, p0, p1 = x & 0xFFFFFFFF, x >> 32, ws & 0xFFFFFFFF, ws >> 32
    qt = x1 * p1 + ((x1 * p0) >> 32) + ((x0 * p1) >> 32)
    assert qt <= M64
    return (x * w - qt * m) & M64


def top_prime_like(bits):
    # any odd modulus just below 2^bits exercises the bounds (primality plays no part in them)
    return (1 << bits) - 59


def test_approximate_product_is_below_4m_and_congruent():
    rng = random.Random(11)
    for bits in (60, 59, 52, 51, 50):
        m = top_prime_like(bits)
        for _ in range(4000):
            w = rng.randrange(m)
            ws = (w << 64) // m
            x = rng.choice([M64, M64 - rng.getrandbits(12), rng.getrandbits(64), rng.getrandbits(40), 16 * m - 1 if 16 * m <= M64 else M64])
            r = approx_product(x, w, ws, m)
            assert r < 4 * m
            assert r % m == (x * w) % m


def _stage(values, m, corrected, rng, forward):
    """One butterfly stage on a list of (value, bound) pairs; returns the new pairs and checks the 64-bit words. Corrected:
    by 8m, a 60-bit prime's forward stage of an even number or inverse stage."""
    out = []
    q4, q8 = 4 * m, 8 * m
    for k in range(0, len(values), 2):
        (X, bx), (Y, by) = values[k], values[k + 1]
        w = rng.randrange(m)
        ws = (w << 64) // m
        if forward:
            if corrected:
                assert max(bx, by) <= 16 * m
                X = X - q8 if X >= q8 else X
                bx = q8
            T = approx_product(Y, w, ws, m)
            assert X + q4 <= M64
            out += [(X + T, bx + q4), (X + q4 - T, bx + q4)]
        else:
            c = q8 if corrected else max(bx, by)
            assert c % m == 0 and by <= c
            S, D = X + Y, X + c - Y
            assert S <= M64 and D <= M64
            if corrected:
                S = S - c if S >= c else S
                out += [(S, c), (approx_product(D, w, ws, m), q4)]
            else:
                out += [(S, 2 * c), (approx_product(D, w, ws, m), q4)]
    for v, b in out:
        assert v < b <= M64 + 1
    return out


def test_forward_ranges():
    rng = random.Random(5)
    for bits, corrected, stages in ((60, True, 16), (52, False, 16), (52, False, 17)):
        m = top_prime_like(bits)
        vals = [(m - 1, m)] * 32          # canonical inputs at the maximum
        for stage in range(stages):
            rng.shuffle(vals)
            vals = _stage(vals, m, corrected and stage % 2 == 0, rng, True)
        bound = max(b for _, b in vals)
        assert bound <= (16 * m if corrected else (1 + 4 * stages) * m)


def test_inverse_ranges():
    rng = random.Random(6)
    # 60-bit primes: inputs below 8q stay below 8q through any number of stages
    m = top_prime_like(60)
    vals = [(8 * m - 1, 8 * m)] * 32
    for _ in range(16):
        rng.shuffle(vals)
        vals = _stage(vals, m, True, rng, False)
    assert max(b for _, b in vals) <= 8 * m
    # primes below 2^52: sums double for the 8 stages of a pass, from inputs below 4q
    m = top_prime_like(52)
    vals = [(4 * m - 1, 4 * m)] * 32
    for _ in range(8):
        vals = sorted(vals, key=lambda vb: -vb[1])    # pair the largest bounds with each other: the worst case
        vals = _stage(vals, m, False, rng, False)
    assert max(b for _, b in vals) <= 1024 * m < (1 << 62)


def test_forward_ranges_with_every_other_stage_corrected():
    """60-bit primes: a stage corrected by 8m takes values below 16m to below 12m, the next one, uncorrected, back to below
    16m <= 2^64; X + T is summed in the product's chain modulo 2^64 and the difference formed from that sum."""
    rng = random.Random(7)
    m = top_prime_like(60)
    assert 16 * m <= 1 << 64
    top = [16 * m - 1, 8 * m, 8 * m - 1, 0, 12 * m]
    vals = [rng.choice(top) for _ in range(64)]
    for stage in range(16):
        limit = 16 * m if stage % 2 == 0 else 12 * m
        rng.shuffle(vals)
        out = []
        for X, Y in zip(vals[::2], vals[1::2]):
            assert X < limit and Y < limit
            w = rng.randrange(m)
            if stage % 2 == 0 and X >= 8 * m:
                X -= 8 * m
            T = approx_product(Y, w, (w << 64) // m, m)
            s = (X + T) & M64
            d = (2 * X + 4 * m - s) & M64
            assert s == X + T and d == X + 4 * m - T
            out += [s, d]
        vals = out
        assert max(vals) < (12 * m if stage % 2 == 0 else 16 * m)
        # a Montgomery product with a canonical word takes the largest value to below 2m
        assert (16 * m - 1) * (m - 1) // (1 << 64) + m <= 2 * m


# ---- double precision: every value an integer of magnitude at most 2^53 (in integers, rounding where the kernels round) ----
def _fp_prime(bits):
    q = (1 << bits) - 1
    while q % 131072 != 1 or any(q % d == 0 for d in (3, 5, 7, 11, 13)):
        q -= 2
    return q


def _fp_reduce(x, q):
    r = x - round(float(x) * (1.0 / q)) * q      # round() of a float: half to even, as the instruction
    assert abs(x) <= 1 << 53
    return r


def _fp_mulmod(a, w, q):
    h = int(float(a * w))
    c = round(float(h) * (1.0 / q))
    assert abs(a) <= 1 << 53 and abs(h - c * q) <= 1 << 53 and abs(a * w - h) <= 1 << 53
    return a * w - c * q


def _fp_stage(top_x, top_y, q, rng, inverse, trials=300):
    """One stage on values up to top_x, top_y (integers) in magnitude, tried at the ends of both ranges: no value passes 2^53
    and each product is within 0.5 + 0.1875 |factor| / q of zero, in units of q."""
    for _ in range(trials):
        X, Y = (rng.choice((-1, 1)) * (t - rng.choice((0, 1, rng.randrange(1 << 20)))) for t in (top_x, top_y))
        w = rng.choice((-1, 1)) * (q // 2 - rng.choice((0, 1, rng.randrange(q // 2))))
        factor = X - Y if inverse else Y
        T = _fp_mulmod(factor, w, q)
        assert abs(T) <= (0.5 + 0.1875 * abs(factor) / q) * q + 2
        for out in (X + Y, T) if inverse else (X + T, X - T):
            assert abs(out) <= 1 << 53


def test_double_precision_forward_ranges():
    """1.1875 A + 0.5 a stage: seven stages from 0.5 q, six from q, five from 1.5 q, four from 2.64 q stay within 2^53. Each
    stage is entered with the bound itself, whatever the sampled values of the one before reached."""
    rng = random.Random(11)
    for bits in (50, 45):
        q = _fp_prime(bits)
        for start, stages in ((0.5, 7), (1.0, 6), (1.5, 5), (2.64, 4)):
            bound = start
            for _ in range(stages):
                _fp_stage(int(bound * q), int(bound * q), q, rng, False)
                bound = 1.1875 * bound + 0.5
                assert bound < 8
        assert ((0.5 * 1.1875 + 0.5) * 1.1875 + 0.5) * 1.1875 + 0.5 < 2.64


def test_double_precision_inverse_ranges():
    """Four stages from 0.5 q end at 8 q < 2^53, their differences at 2 q; from q the round of four does so too if the two
    sums of eight values are reduced before its last stage."""
    rng = random.Random(12)
    q = _fp_prime(50)
    for bound in (0.5, 1.0, 2.0, 4.0):
        assert 2 * bound * q <= 1 << 53 and 0.5 + 0.1875 * 2 * bound <= 2
        _fp_stage(int(bound * q), int(bound * q), q, rng, True)
    # the 16 values of a round from q, bounds in units of q
    x = [1.0] * 16
    for half in (1, 2, 4, 8):
        if half == 8:
            assert x[0] == x[8] == 8
            for at in (0, 8):
                assert abs(_fp_reduce(int(x[at] * q), q)) <= q // 2 + 1
                x[at] = 0.5
        for g in range(0, 16, 2 * half):
            for p in range(g, g + half):
                s = x[p] + x[p + half]
                assert s <= 8
                _fp_stage(int(x[p] * q), int(x[p + half] * q), q, rng, True, 30)
                x[p], x[p + half] = s, 0.5 + 0.1875 * s


def test_centred_representative_by_rounding():
    """x - rint(x / q) q is the centred representative for |x| <= q, up to its ends."""
    for bits in (50, 49, 40):
        q = _fp_prime(bits)
        h = (q - 1) // 2
        for x in (0, 1, h - 1, h, h + 1, h + 2, q - 1, q):
            for v in (x, -x):
                r = _fp_reduce(v, q)
                assert (r - v) % q == 0 and abs(r) <= h


def test_conversion_of_eight_double_precision_sources():
    """H + L of eight products of 2^98, reduced with one rounded quotient: exact, at most 1.3 q."""
    rng = random.Random(13)
    for bits in (50, 40):
        q, M = _fp_prime(bits), 3 << 101
        for _ in range(200):
            H, L, want = M, 0, 0
            for _ in range(8):
                y = rng.choice((-1, 1)) * ((1 << 49) - 1 - rng.choice((0, rng.randrange(1 << 48))))
                c = rng.choice((1, 1, -1)) * (q // 2 - rng.choice((0, rng.randrange(q // 2))))
                want += y * c
                Hn = int(float(H + y * c))
                L += y * c - (Hn - H)
                H = Hn
                assert abs(L) <= 1 << 53
            h = H - M
            t = round(float(L * (1.0 / q) + float(h) * (1.0 / q)))
            assert abs(h - t * q) <= 1 << 53
            x = h - t * q + L
            assert (x - want) % q == 0 and abs(x) <= 1.3 * q


def test_inverse_ranges_with_products_left_alone():
    """60-bit primes: sums corrected by 8m stay below 8m; the sum of two products (below 4m) needs no correction."""
    rng = random.Random(14)
    m = top_prime_like(60)
    for start in (8 * m - 1, m - 1):
        x = [rng.choice((start, start - rng.randrange(start), 0)) for _ in range(16)]
        for half in (1, 2, 4, 8):
            for g in range(0, 16, 2 * half):
                for p in range(half):
                    X, Y, w = x[g + p], x[g + p + half], rng.randrange(m)
                    products = bool(p & (half >> 1))
                    assert max(X, Y) < (4 * m if products else 8 * m)
                    S, D = X + Y, X + (4 if products else 8) * m - Y
                    assert 0 < D <= M64 and S <= M64
                    if not products and S >= 8 * m:
                        S -= 8 * m
                    T = approx_product(D, w, (w << 64) // m, m)
                    assert S < 8 * m and T < 4 * m
                    assert (S - X - Y) % m == 0 and (T - w * (X - Y)) % m == 0
                    x[g + p], x[g + p + half] = S, T


def test_montgomery_product_by_words():
    """x < 2^63, e and m below 2^60: two 32-bit Montgomery words whose middle sum, with both carries, fits 64 bits."""
    rng = random.Random(15)
    M32 = (1 << 32) - 1
    for bits in (60, 53, 50):
        m = top_prime_like(bits)
        mi = -pow(m, -1, 1 << 32) & M32
        m0, m1 = m & M32, m >> 32
        for _ in range(3000):
            x = rng.choice(((1 << 63) - 1, min(8 * m, 1 << 63) - 1, rng.getrandbits(63)))
            e = rng.choice((m - 1, rng.randrange(m)))
            x0, x1, e0, e1 = x & M32, x >> 32, e & M32, e >> 32
            p = x0 * e0
            mid = x0 * e1 + (x1 * e0 + (p >> 32))
            assert mid <= M64
            u0 = (p & M32) * mi & M32
            v0 = u0 * m0 + (p & M32)
            assert v0 <= M64 and v0 & M32 == 0
            mid = u0 * m1 + mid + (v0 >> 32)
            assert mid <= M64
            u1 = (mid & M32) * mi & M32
            v1 = u1 * m0 + (mid & M32)
            r = x1 * e1 + (u1 * m1 + (mid >> 32)) + (v1 >> 32)
            assert v1 <= M64 and v1 & M32 == 0 and r <= M64
            assert (r * (1 << 64) - x * e) % m == 0
            assert r <= x * e // (1 << 64) + m
            if x < 8 * m:
                assert r < 2 * m


def _narrow_ok(n, bs, bt, bt_min):
    """The host's rule for three sums of 30-bit partial products: n sources below 2^bs, targets below 2^bt, at least 2^(bt_min - 1)."""
    if bs > 60 or bt > 60 or bt_min < 36:
        return False
    w, y1, c1 = (1 << 30) - 1, 1 << max(0, bs - 30), 1 << max(0, bt - 30)
    amax = n * w * w + n * w + w * w
    bmax = n * (w * c1 + y1 * w) + n * c1 + (1 << 34) + w * c1 + w * w
    cmax = n * y1 * c1 + (1 << 34) + w * c1 + w * w
    return max(amax, bmax, cmax) < 1 << 64


def _odd_below(bits):
    return (1 << bits) - 59


def _redc60(sums, m):
    """Two words of the base-2^30 Montgomery reduction of a + b 2^30 + c 2^60; no word may pass 2^64."""
    M30 = (1 << 30) - 1
    a, b, c = sums
    q0, q1, qi = m & M30, m >> 30, -pow(m, -1, 1 << 30) & M30
    u = (a & M30) * qi & M30
    a += u * q0
    assert a <= M64 and a & M30 == 0
    b += (a >> 30) + u * q1
    assert b <= M64
    u = (b & M30) * qi & M30
    b += u * q0
    assert b <= M64 and b & M30 == 0
    c += (b >> 30) + u * q1
    assert c <= M64
    return c


def test_conversion_of_split_sources():
    """At most 8 sources: V / 2^60 modulo m below V / 2^60 + m <= 9m. To a double-precision target the result goes through
    an offset, 2^62 - 4m in the top sum: what is left of it after subtracting 2^62 is exact in doubles and below 2^53."""
    rng = random.Random(16)
    M30, tried = (1 << 30) - 1, 0
    for bs in (60, 55, 51, 50, 36, 30):
        for bt in (60, 52, 50, 45, 36):
            for n in range(1, 9):
                if not _narrow_ok(n, bs, bt, bt):
                    continue
                tried += 1
                m = _odd_below(bt)
                for trial in range(20):
                    worst = trial % 2 == 0
                    ys = [(1 << bs) - 1 if worst else rng.getrandbits(bs) for _ in range(n)]
                    cs = [m - 1 if worst else rng.randrange(m) for _ in range(n)]
                    off = m - 1 if worst else rng.randrange(m)
                    V = off + sum(y * c for y, c in zip(ys, cs))
                    a, b, c = off & M30, off >> 30, 0
                    for y, k in zip(ys, cs):
                        a += (y & M30) * (k & M30)
                        b += (y & M30) * (k >> 30) + (y >> 30) * (k & M30)
                        c += (y >> 30) * (k >> 30)
                    assert max(a, b, c) <= M64
                    r = _redc60((a, b, c), m)
                    assert (r * (1 << 60) - V) % m == 0 and r <= V // (1 << 60) + m and r < 9 * m
                    if bt <= 50:
                        v = _redc60((a, b, c + (1 << 62) - 4 * m), m)
                        assert v == r + (1 << 62) - 4 * m and -4 * m <= v - (1 << 62) < 5 * m <= 1 << 53
                        hi, lo = 2.0 ** 84 + 2.0 ** 32 * (v >> 32), 2.0 ** 52 + (v & 0xFFFFFFFF)
                        assert int(hi) == (1 << 84) + (v >> 32 << 32)
                        big = 2.0 ** 84 + 2.0 ** 62 + 2.0 ** 52
                        assert int(big) == (1 << 84) + (1 << 62) + (1 << 52)
                        x = (hi - big) + lo
                        assert int(x) == v - (1 << 62)
                        assert abs(_fp_reduce(int(x), m)) <= m // 2
    assert tried > 150


def _redc90(sums, m):
    """Three words of the base-2^30 Montgomery reduction of a + b 2^30 + c 2^60; no word may pass 2^64."""
    M30 = (1 << 30) - 1
    a, b, c = sums
    q0, q1, qi = m & M30, m >> 30, -pow(m, -1, 1 << 30) & M30
    u = (a & M30) * qi & M30
    a += u * q0
    assert a <= M64 and a & M30 == 0
    b += (a >> 30) + u * q1
    assert b <= M64
    u = (b & M30) * qi & M30
    b += u * q0
    assert b <= M64 and b & M30 == 0
    c += (b >> 30) + u * q1
    assert c <= M64
    u = (c & M30) * qi & M30
    c += u * q0
    assert c <= M64 and c & M30 == 0
    return (c >> 30) + u * q1


def test_endings_of_the_separate_conversions():
    """At most 8 sources, and the sources above half their modulus times one constant: in three sums V / 2^90 modulo m below
    m + 2^34, in four sums V / 2^64 below 2m, so that one subtraction ends both."""
    rng = random.Random(16)
    M30, tried = (1 << 30) - 1, 0
    for bs in (60, 55, 51, 50, 36, 30):
        for bt in (60, 52, 50, 45, 36, 30):
            for n in range(1, 9):
                tried += _narrow_ok(n, bs, bt, bt)
                m = _odd_below(bt)
                for trial in range(20):
                    worst = trial % 2 == 0
                    ys = [(1 << bs) - 1 if worst else rng.getrandbits(bs) for _ in range(n)]
                    cs = [m - 1 if worst else rng.randrange(m) for _ in range(n)]
                    count, neg = (n, m - 1) if worst else (rng.randint(0, n), rng.randrange(m))
                    V = count * neg + sum(y * c for y, c in zip(ys, cs))
                    s00, s01, s10, s11 = count * (neg & M30), count * (neg >> 30), 0, 0
                    for y, k in zip(ys, cs):
                        s00 += (y & M30) * (k & M30)
                        s01 += (y & M30) * (k >> 30)
                        s10 += (y >> 30) * (k & M30)
                        s11 += (y >> 30) * (k >> 30)
                    assert max(s00, s01, s10, s11) <= M64
                    assert V == s00 + ((s01 + s10) << 30) + (s11 << 60) and V < 1 << 128
                    u = (V & M64) * (-pow(m, -1, 1 << 64) & M64) & M64
                    r = (V + u * m) >> 64
                    assert (r * (1 << 64) - V) % m == 0 and r < 2 * m
                    if _narrow_ok(n, bs, bt, bt):
                        assert s01 + s10 <= M64
                        r = _redc90((s00, s01 + s10, s11), m)
                        assert (r * (1 << 90) - V) % m == 0 and r < min(m + (1 << 34), 2 * m)
    assert tried > 150


def test_integer_inner_sums_carry_into_their_top_word():
    """Four sums of 30-bit partial products, settled after every 11 terms: nothing passes 2^64, the value modulo m stays, the
    top sum returns below 4m and the others below 2^30."""
    M30 = (1 << 30) - 1
    rng = random.Random(17)
    for m in (_odd_below(60), _odd_below(52), _odd_below(50), _odd_below(30), _odd_below(20)):
        mu = (1 << 64) // m
        for worst in (True, False):
            s00 = s01 = s10 = s11 = want = 0
            for k in range(1, 45):
                x, c = (m - 1, m - 1) if worst else (rng.randrange(m), rng.randrange(m))
                want += x * c
                s00 += (x & M30) * (c & M30)
                s01 += (x & M30) * (c >> 30)
                s10 += (x >> 30) * (c & M30)
                s11 += (x >> 30) * (c >> 30)
                assert max(s00, s01, s10, s11) <= M64
                if k % 11 == 0:
                    s01 += s00 >> 30
                    assert s01 <= M64
                    s11 += (s01 >> 30) + (s10 >> 30)
                    assert s11 <= M64
                    s00, s01, s10 = s00 & M30, s01 & M30, s10 & M30
                    x0, x1, p0, p1 = s11 & 0xFFFFFFFF, s11 >> 32, mu & 0xFFFFFFFF, mu >> 32
                    qt = x1 * p1 + (x1 * p0 >> 32) + (x0 * p1 >> 32)
                    s11 -= qt * m
                    assert 0 <= s11 < 4 * m
                V = s00 + ((s01 + s10) << 30) + (s11 << 60)
                assert V < 1 << 128 and (V - want) % m == 0
        # the highest a term-by-term argument can reach: a settled value and 11 products of the largest halves
        assert 11 * M30 * M30 + M30 + (1 << 34) <= M64 and 11 * M30 * M30 + 4 * _odd_below(60) + (1 << 36) <= M64


def test_double_precision_inner_sums_in_two_parts():
    """Products of a residue and a centred word added to H in the binade of 1.5 * 2^103, what that rounds off to L, both folded
    into L after every fifth: exact, at most 1.45 q after a fold, below 7.9 * 2^50 throughout."""
    rng = random.Random(18)
    for bits in (50, 49, 40, 30):
        q, M = _fp_prime(bits), 3 << 102
        half, qinv = (q - 1) // 2, 1.0 / q
        for x_of, c_of in ((lambda: q - 1, lambda: q - 1), (lambda: q - 1, lambda: 0),
                           (lambda: rng.choice((q - 1, rng.randrange(q))), lambda: rng.choice((0, q - 1, rng.randrange(q))))):
            H, L, sx, want = M, 0, 0, 0
            for k in range(1, 41):
                x, c = x_of(), c_of()
                want += x * c
                sx += x
                p = x * (c - half)
                Hn = int(float(H + p))
                assert 1 << 103 <= Hn < 1 << 104
                rest = p - (Hn - H)
                assert abs(rest) <= 1 << 50
                L, H = L + rest, Hn
                assert abs(L) <= 7.9 * 2 ** 50 and sx <= 1 << 53
                if k % 5 == 0 or k == 40:
                    h = H - M
                    t = round(float(Fraction(L) * Fraction(qinv) + Fraction(float(h) * qinv)))   # one fma
                    r = h - t * q
                    assert abs(r) <= 1 << 53 and int(float(h)) == h
                    L, H, sx = r + L, M, _fp_reduce(sx, q)
                    assert abs(L) <= 1.45 * q
            total = L + _fp_mulmod(sx, half, q)
            assert abs(_fp_reduce(total, q)) <= q // 2 + 1 and (total - want) % q == 0


def test_unreduced_digits_of_the_fused_inner_product():
    """A round of four stages from q/2 is left as it is, at most 3.64 q; its product with a key word is at most 1.87 q, and
    four of them with a folded sum stay below 8 q."""
    rng = random.Random(19)
    q = _fp_prime(50)
    bound = 0.5
    for _ in range(4):
        bound = 1.1875 * bound + 0.5
    assert bound <= 3.64
    largest = 0.5 + 0.375 * 3.64
    assert largest <= 1.87 and 4 * 1.87 + 0.5 < 8
    top = int(3.64 * q)
    for _ in range(100):
        acc = rng.choice((-1, 1)) * (q // 2)
        for k in range(4):
            x = rng.choice((-1, 1)) * (top - rng.choice((0, 1, rng.randrange(1 << 20))))
            T = _fp_mulmod(x, q - 1 - rng.choice((0, rng.randrange(1 << 20))), q)
            assert abs(T) <= 1.87 * q
            acc += T
            assert abs(acc) <= 1 << 53
        assert abs(_fp_reduce(acc, q)) <= q // 2 + 1
    # and at the bound itself, which sampled products do not reach
    for sign in (-1, 1):
        assert abs(_fp_reduce(sign * int((4 * 1.87 + 0.5) * q), q)) <= q // 2 + 1
