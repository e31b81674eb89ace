"""GPU parity on chains whose primes differ in size (a 60-bit first prime before 50-bit ones, a 50-bit special prime beside
60-bit ones): both arithmetic kinds among the main limbs, digits and sums over both, on every kind of ring."""
import pytest

import test_gpu_two_pass_rings as calls
from ckks_inputs import galois_element, uniform_residues
from ckks_inputs.params import CkksParams, find_ntt_primes, find_psi
from oracle import ref

pytestmark = pytest.mark.gpu


def mixed_params(logN, q_bits, p_bits, dnum):
    primes = []
    for bits in q_bits + p_bits:
        primes += find_ntt_primes(bits, 1, logN, exclude=set(primes))
    q, p = primes[:len(q_bits)], primes[len(q_bits):]
    return CkksParams(logN=logN, q=q, p=p, dnum=dnum, psi=[find_psi(m, logN) for m in primes])


SHAPES = [
    # logN, sizes of the main primes, of the special primes, dnum, nlimbs, B
    (11, [60, 50], [60], 2, 2, 1),
    (12, [60, 50, 50, 50], [60, 60], 2, 4, 2),
    (12, [50, 60, 50], [50, 60], 1, 3, 1),
    (13, [60, 50, 50, 50], [60, 50], 2, 4, 2),
    (15, [60, 50, 50], [60], 3, 3, 2),
    (14, [50, 55, 50, 51], [60, 60], 2, 3, 1),   # all three classes
    (16, [60, 50, 50], [60, 60], 2, 3, 2),
]


@pytest.mark.parametrize("logN,q_bits,p_bits,dnum,nl,B", SHAPES)
def test_calls_on_mixed_primes(logN, q_bits, p_bits, dnum, nl, B, monkeypatch):
    p = mixed_params(logN, q_bits, p_bits, dnum)
    monkeypatch.setattr(calls, "make_params", lambda *shape: p)
    calls.test_calls_on_the_smaller_two_pass_rings((), nl, B)


def test_extended_basis_calls_on_mixed_primes():
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = mixed_params(16, [60, 50, 50], [60, 50], 2)
    rc, gc, nl, B, n1, n2 = ref.RefContext(p), gpu.Context(p), 3, 2, 2, 2
    ct = uniform_residues(1, p.q, (B, 2), p.N)
    keys = [uniform_residues(2 + i, p.moduli, (p.dnum, 2), p.N) for i in range(3)]
    gs = [galois_element(k, p.logN) for k in (1, 5, 9)]
    d_ct, d_keys = to_dev(ct), [to_dev(k) for k in keys]
    out = torch.empty_like(d_ct)
    gpu.ckks_hrot_sum(gc, out, d_ct, B, nl, gs, d_keys, gc.workspace(gpu.OP_HROT_SUM, B, nl))
    assert_same(to_host(out), rc.hrot_sum(ct, gs, keys), "hrot_sum")
    pt = uniform_residues(7, p.moduli, (n2, n1), p.N)
    gpu.ckks_pcmm_bsgs_double_hoisted(gc, out, d_ct, B, nl, to_dev(pt), n1, n2, 1, d_keys[:1], d_keys[1:2],
                                      gc.workspace(gpu.OP_PCMM_BSGS_DH, B, nl, n1))
    assert_same(to_host(out), rc.pcmm_bsgs_double_hoisted(ct, pt, n1, n2, 1, keys[:1], keys[1:2]), "double-hoisted")
    gc.close()
