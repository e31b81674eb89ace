"""GPU parity of the base conversion fused with the row passes around it, where its instantiations differ: source counts
around 4, 6 and 8, the separate kernels beyond, each arithmetic kind on either side, short digits, shares of the targets."""
import pytest

import test_gpu_two_pass_rings as calls

gpu_only = pytest.mark.gpu

SHAPES = [
    # (logN nq qbits np pbits dnum), nlimbs, B
    ((13, 4, 50, 4, 60, 1), 4, 2),
    ((13, 6, 50, 5, 60, 1), 6, 1),
    ((14, 8, 45, 8, 60, 1), 7, 2),     # a digit one limb short
    ((15, 7, 50, 6, 60, 1), 7, 1),
    ((13, 9, 50, 9, 60, 1), 9, 1),     # one source more than the fused kernel takes
    ((13, 8, 60, 8, 60, 1), 8, 1),     # 60-bit primes on both sides: the general reduction
    ((14, 4, 51, 4, 60, 1), 4, 2),     # 51-bit sources
    ((13, 6, 50, 3, 50, 2), 6, 2),     # double precision on both sides, special primes too
    ((13, 3, 30, 2, 50, 2), 3, 40),    # 30-bit targets: the general reduction, which keeps the separate kernels
]


@gpu_only
@pytest.mark.parametrize("shape,nl,B", SHAPES)
def test_calls_around_the_fused_conversion(shape, nl, B):
    calls.test_calls_on_the_smaller_two_pass_rings(shape, nl, B)


def _kernels_of(gpu, gc, call):
    gpu.ckks_prof_reset(gc)
    gpu.ckks_prof_enable(gc, True)
    call()
    gpu.ckks_prof_enable(gc, False)
    return {k: n for k, (ms, n) in gpu.ckks_prof_collect(gc).items()}


@gpu_only
@pytest.mark.parametrize("shape,B,alone", [
    # (logN nq qbits np pbits dnum), B, whether the sources' inverse row pass runs in a kernel of its own
    ((13, 6, 50, 2, 60, 3), 96, False),    # one share a tile: a workgroup walks over all targets of both kinds
    ((13, 6, 60, 2, 50, 3), 96, False),    # the same from integer sources
    ((13, 6, 50, 3, 50, 2), 96, False),
    ((14, 14, 50, 7, 60, 2), 32, False),   # seven sources
    ((15, 6, 50, 3, 60, 2), 20, False),
    ((15, 12, 60, 6, 50, 2), 16, False),
    ((14, 6, 50, 2, 60, 3), 24, False),    # shares of a few targets
    ((14, 14, 50, 7, 60, 2), 1, True),
    ((13, 12, 60, 6, 50, 2), 2, True),
])
def test_shares_of_the_targets(shape, B, alone):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import galois_element, make_params, uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = make_params(*shape)
    rc, gc, nl = ref.RefContext(p), gpu.Context(p), len(p.q)
    ct, ct2 = (uniform_residues(40 + i, p.q, (B, 2), p.N) for i in range(2))
    evk, g, some = uniform_residues(42, p.moduli, (p.dnum, 2), p.N), galois_element(9, p.logN), sorted({0, B // 2, B - 1})
    d_ct, d_ct2, d_evk = to_dev(ct), to_dev(ct2), to_dev(evk)
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_HROT, B, nl)
    ran = _kernels_of(gpu, gc, lambda: gpu.ckks_hrot(gc, out, d_ct, B, nl, g, d_evk, ws))
    assert ran["conv_rows_kernel"] == 2, ran
    assert any(k.startswith("ntt16_inv_rows") for k in ran) == alone, ran
    assert_same(to_host(out)[some], rc.hrot(ct[some], g, evk), "hrot")
    gpu.ckks_hmult_relin(gc, out, d_ct, d_ct2, B, nl, d_evk, ws)
    assert_same(to_host(out)[some], rc.hmult_relin(ct[some], ct2[some], evk), "hmult_relin")
    gc.close()


def test_double_precision_conversion_is_exact_at_its_bounds():
    """The recurrence of the conversion of double-precision sources, in correctly rounded double arithmetic: the running sum
    stays in its binade, both parts are exact, and what one quotient of their sum leaves is congruent and at most 1.3 moduli."""
    import random
    from fractions import Fraction

    def rnd(x):   # one rounding to double, ties to even, as the hardware's fma and add do
        return float(x)
    M, rng = 1.5 * 2.0 ** 102, random.Random(3)
    top = (1 << 50) - 27     # the largest sources and targets (primality plays no part in the bounds)
    for trial in range(300):
        n = rng.choice([1, 4, 8])
        q = rng.choice([top, top, (1 << 40) - 87, (1 << 20) + 7])
        sign = rng.choice([1, -1])
        if trial % 3:
            ys = [rng.randint(-(top // 2), top // 2) for _ in range(n)]
            cs = [rng.randint(-(q // 2), q // 2) for _ in range(n)]
        else:                # every product at the largest magnitude, all of one sign
            ys, cs = [sign * (top // 2)] * n, [q // 2] * n
        H, L = M, 0.0
        for y, c in zip(ys, cs):
            Hn = rnd(Fraction(y) * c + Fraction(H))
            assert 2.0 ** 102 <= Hn < 2.0 ** 103
            h = Hn - H
            assert Fraction(h) == Fraction(Hn) - Fraction(H)
            rest = Fraction(y) * c - Fraction(h)
            assert abs(rest) <= 2 ** 49 and Fraction(rnd(rest)) == rest
            assert Fraction(L) + rest == Fraction(L + float(rest))
            H, L = Hn, L + float(rest)
        total, h, qinv = sum(y * c for y, c in zip(ys, cs)), H - M, 1.0 / q
        assert Fraction(h) + Fraction(L) == total
        t = round(rnd(Fraction(L) * Fraction(qinv) + Fraction(h * qinv)))
        r = Fraction(h) - Fraction(t) * q
        assert Fraction(rnd(r)) == r
        out = rnd(r) + L
        assert Fraction(out) == r + Fraction(L)
        assert (Fraction(out) - total) % q == 0 and abs(out) <= 1.3 * q


@gpu_only
@pytest.mark.parametrize("shape,nl,B,R", [
    ((16, 5, 50, 2, 60, 5), 5, 6, 3),      # five digits: the kernel for any number; two groups of three; 15 products
    ((16, 4, 50, 2, 60, 4), 4, 5, 9),      # four digits, two groups with one place empty
    ((16, 3, 50, 1, 50, 3), 2, 3, 2),      # double-precision special primes
    ((16, 4, 60, 2, 60, 4), 4, 3, 30),     # integer main primes: 150 products, sums reduced on the way
    ((16, 2, 50, 1, 60, 2), 2, 10, 2),     # a group of four and two of three
    ((16, 2, 50, 1, 60, 1), 2, 7, 4),      # four and three, one digit
    ((16, 2, 50, 1, 60, 2), 2, 5, 3),      # two positions of one ciphertext per lane
    ((16, 5, 50, 1, 60, 5), 5, 1, 3),
    ((16, 2, 60, 2, 60, 2), 2, 2, 1),      # one rotation, integer main primes
    ((16, 2, 60, 2, 60, 2), 2, 2, 8),      # 16 products an output: partial products
    ((16, 2, 50, 2, 60, 1), 2, 3, 65),     # one rotation beyond an argument table
])
def test_hoisted_sums_of_several_ciphertexts(shape, nl, B, R):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import galois_element, make_params, uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = make_params(*shape)
    rc, gc = ref.RefContext(p), gpu.Context(p)
    ct = uniform_residues(1, p.q[:nl], (B, 2), p.N)
    ct[0] = [[[m - 1] for m in p.q[:nl]]] * 2
    keys = [uniform_residues(2 + r, p.moduli, (p.dnum, 2), p.N) for r in range(min(R, 3))]
    keys[0][:] = [[[[m - 1] for m in p.moduli]]]
    evks, gs = [keys[r % 3] for r in range(R)], [galois_element(5 * r + 1, p.logN) for r in range(R)]
    d_keys = [to_dev(k) for k in keys]
    out = torch.empty((B, 2, nl, p.N), dtype=torch.int64, device="cuda")
    gpu.ckks_hrot_sum(gc, out, to_dev(ct), B, nl, gs, [d_keys[r % 3] for r in range(R)], gc.workspace(gpu.OP_HROT_SUM, B, nl))
    assert_same(to_host(out), rc.hrot_sum(ct, gs, evks), "hrot_sum")
    gc.close()
