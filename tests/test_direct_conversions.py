"""Conversions of at most 6 double-precision sources where every prime is double precision: on the vector units, exact sums in two
doubles. Which kernels a call takes is read off its launches without a GPU; on it the calls are compared with the oracle."""
import pytest

import test_gpu_two_pass_rings as calls
from test_gpu_mixed_primes import mixed_params

SHAPES = [
    # logN, sizes of the main primes, of the special primes, dnum; nlimbs, B; sources of the kernels of ModUp and ModDown (0: bytes)
    ((13, [50] * 2, [50], 2), 2, 32, 4, 4),
    ((14, [50, 45, 40, 50], [50] * 4, 1), 4, 3, 4, 4),
    ((15, [50] * 5, [50, 40, 30], 2), 4, 2, 4, 4),           # a digit of one limb; special primes below the main ones
    ((13, [30] * 5, [50] * 5, 1), 5, 1, 6, 6),
    ((14, [50] * 9, [50] * 5, 2), 8, 2, 6, 6),               # three of five limbs in the last digit
    ((15, [50] * 12, [50] * 6, 2), 12, 1, 6, 6),             # the inverse row pass before the shares
    ((16, [50] * 6, [50] * 6, 1), 6, 1, 6, 6),
    ((16, [50] * 4, [50], 4), 3, 5, 4, 4),
    ((13, [50] * 6, [50] * 7, 1), 6, 2, 6, 0),
    ((13, [50] * 7, [50] * 6, 1), 7, 2, 0, 6),
    ((13, [50] * 4, [50, 50, 50, 60], 1), 4, 2, 0, None),    # an integer-class prime among them (ModDown: kernels of its own)
    ((13, [50] * 4, [60] * 2, 2), 4, 2, 0, 0),
]


def _form(kernel):
    return next((n for n in (4, 6) if "ELi%dELb1E" % n in kernel and "ELb1EEv" in kernel), 0)


@pytest.mark.parametrize("shape,nl,B,up,down", SHAPES)
def test_route(shape, nl, B, up, down):
    from launch_trace import trace
    kernels = [name for what, _, name in trace(shape, {}, nl, B, ["hrot"]) if what == "launch" and "conv_rows_kernel" in name
               and "bconv" not in name]
    assert [_form(k) for k in kernels] == [n for n in (up, down) if n is not None], kernels


def test_route_without_double_precision_bodies():
    from launch_trace import trace
    kernels = [name for what, _, name in trace(SHAPES[1][0], {1: 1}, 4, 2, ["hrot"]) if what == "launch" and "conv_rows" in name]
    assert kernels and not any(_form(k) for k in kernels)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,nl,B,up,down", SHAPES)
def test_calls(shape, nl, B, up, down, monkeypatch):
    p = mixed_params(*shape)
    monkeypatch.setattr(calls, "make_params", lambda *s: p)
    calls.test_calls_on_the_smaller_two_pass_rings((), nl, B)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,nl,B", [s[:3] for s in SHAPES[1:6]])
def test_residues_at_the_ends_of_their_range(shape, nl, B):
    """Sources around half of their prime and at its ends."""
    import numpy as np
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import galois_element, uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(*shape)
    rc, gc = ref.RefContext(p), gpu.Context(p)
    rng = np.random.default_rng(4)
    ct = np.empty((B, 2, nl, p.N), dtype=np.uint64)
    alpha = -(-len(p.q) // p.dnum)
    for i, q in enumerate(p.q[:nl]):
        lo, scale = i // alpha * alpha, 1   # the source is the residue times the inverse of this
        for k in range(lo, min(lo + alpha, nl)):
            scale = scale * (p.q[k] if k != i else 1) % q
        ends = [v * scale % q for v in (0, 1, q // 2, q // 2 + 1, q - 1)]
        ct[:, :, i] = rng.choice(np.array(ends, dtype=np.uint64), (B, 2, p.N))
    ct = rc.ntt(ct, list(range(nl)))
    evk, g = uniform_residues(7, p.moduli, (p.dnum, 2), p.N), galois_element(5, p.logN)
    d = to_dev(ct)
    out = torch.empty_like(d)
    gpu.ckks_hrot(gc, out, d, B, nl, g, to_dev(evk), gc.workspace(gpu.OP_HROT, B, nl))
    assert_same(to_host(out), rc.hrot(ct, g, evk), "hrot")
    gc.close()
