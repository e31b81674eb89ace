"""GPU parity of the few-launch key switch of the ring 2^12: every modulus class, both conversion reductions, more
sources than one chunk of a conversion, ragged digits and levels, more ciphertexts than one argument table; bit-exact."""
import numpy as np
import pytest

import test_gpu_two_pass_rings as calls
from ckks_inputs import galois_element, make_params, uniform_residues
from oracle import ref

pytestmark = pytest.mark.gpu

SHAPES = [
    # (logN nq qbits np pbits dnum), nlimbs, B
    ((12, 4, 40, 1, 50, 2), 4, 3),     # double precision throughout
    ((12, 5, 50, 2, 60, 3), 5, 1),     # digits 2, 2, 1; Harvey bodies on the special limbs
    ((12, 5, 50, 2, 60, 3), 3, 2),
    ((12, 3, 51, 2, 51, 2), 3, 2),     # uncorrected integer bodies throughout
    ((12, 8, 60, 8, 60, 1), 8, 2),     # eight 60-bit sources: the general reduction
    ((12, 17, 50, 16, 60, 1), 17, 1),  # conversions in two chunks
]


@pytest.mark.parametrize("shape,nl,B", SHAPES)
def test_calls_on_the_whole_limb_ring(shape, nl, B):
    calls.test_calls_on_the_smaller_two_pass_rings(shape, nl, B)


def test_rotations_beyond_one_argument_table():
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = make_params(12, 3, 50, 1, 60, 3)
    gc, B, nl = gpu.Context(p), 66, 3
    gs = [galois_element(3 * b + 1, p.logN) for b in range(B)]
    d_ct = to_dev(uniform_residues(5, p.q, (B, 2), p.N))
    keys = [to_dev(uniform_residues(6 + b, p.moduli, (p.dnum, 2), p.N)) for b in range(3)]
    out, one = torch.empty_like(d_ct), torch.empty_like(d_ct[:1])
    ws = gc.workspace(gpu.OP_HROT, B, nl)
    gpu.ckks_hrot_multi(gc, out, d_ct, B, nl, gs, [keys[b % 3] for b in range(B)], ws)
    for b in (0, 63, 64, 65):
        gpu.ckks_hrot(gc, one, d_ct[b:b + 1].contiguous(), 1, nl, gs[b], keys[b % 3], ws)
        assert_same(to_host(out)[b:b + 1], to_host(one), "ciphertext %d" % b)
    gc.close()


def test_large_batches_of_many_limbs_go_by_steps():
    """From the size where rereading sources costs more than launches, one kernel per step; the same bits either way."""
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = make_params(12, 16, 50, 4, 60, 4)
    rc, gc, B, nl = ref.RefContext(p), gpu.Context(p), 39, 16     # 39 x 4 digits x 20 limbs
    ct, ct2 = (uniform_residues(20 + i, p.q, (B, 2), p.N) for i in range(2))
    evk, g, some = uniform_residues(22, p.moduli, (p.dnum, 2), p.N), galois_element(11, p.logN), [0, B - 1]
    pt = uniform_residues(23, p.q, (2, 1), p.N)
    d_ct, d_ct2, d_evk, d_pt = to_dev(ct), to_dev(ct2), to_dev(evk), to_dev(pt)
    d3 = torch.empty((B, 3, nl, p.N), dtype=torch.int64, device="cuda")
    gpu.ckks_tensor_acc(gc, d3, d_ct, d_ct2, None, B, nl)
    d = d_ct[:, 1].contiguous()

    def calls(idx):
        n, pick = len(idx), lambda t: t[idx].contiguous()
        out = torch.empty_like(d_ct[:n])
        ws, wsp = gc.workspace(gpu.OP_HROT, n, nl), gc.workspace(gpu.OP_PCMM_BSGS, n, nl, 1)
        yield "hrot", lambda: gpu.ckks_hrot(gc, out, pick(d_ct), n, nl, g, d_evk, ws), out
        yield "hrot_add", lambda: gpu.ckks_hrot_add(gc, out, pick(d_ct), pick(d_ct2), n, nl, g, d_evk, ws), out
        yield "keyswitch", lambda: gpu.ckks_keyswitch(gc, out, pick(d), n, nl, d_evk, 0, p.dnum, ws), out
        yield "relin", lambda: gpu.ckks_relin(gc, out, pick(d3), n, nl, d_evk, ws), out
        yield "hmult", lambda: gpu.ckks_hmult_relin(gc, out, pick(d_ct), pick(d_ct2), n, nl, d_evk, ws), out
        yield "pcmm", lambda: gpu.ckks_pcmm_bsgs(gc, out, pick(d_ct), n, nl, d_pt, 1, 2, 1, [], [d_evk], wsp), out

    def results(idx, kernel):
        for name, run, out in calls(idx):
            gpu.ckks_prof_reset(gc)
            gpu.ckks_prof_enable(gc, True)
            run()
            gpu.ckks_prof_enable(gc, False)
            assert gpu.ckks_prof_collect(gc).get(kernel, (0, 0))[1] > 0, "%s of %d without %s" % (name, len(idx), kernel)
            yield name, to_host(out)
    few = dict((name, r) for name, r in results(some, "ks12_final_kernel"))
    for name, got in results(list(range(B)), "modup_kernel"):
        assert_same(got[some], few[name], name)
    assert_same(few["hrot"], rc.hrot(ct[some], g, evk), "hrot")
    assert_same(few["hmult"], rc.hmult_relin(ct[some], ct2[some], evk), "hmult")
    assert_same(few["pcmm"], rc.pcmm_bsgs(ct[some], pt, 1, 2, 1, [], [evk]), "pcmm")
    # a key per ciphertext stays in one sequence
    gpu.ckks_prof_reset(gc)
    gpu.ckks_prof_enable(gc, True)
    out = torch.empty_like(d_ct)
    gpu.ckks_hrot_multi(gc, out, d_ct, B, nl, [g] * B, [d_evk] * B, gc.workspace(gpu.OP_HROT, B, nl))
    gpu.ckks_prof_enable(gc, False)
    assert gpu.ckks_prof_collect(gc)["ks12_final_kernel"][1] == 1
    assert_same(to_host(out)[some], few["hrot"], "hrot_multi")
    gc.close()
