"""GPU parity of the two-pass kernels on the rings 2^13 .. 2^15 (2^16 has its own tests): every modulus class, key
switching in all its forms, ragged digits and levels, group counts that are no multiple of 8; bit-exact."""
import numpy as np
import pytest

from ckks_inputs import galois_element, make_params, uniform_residues
from oracle import ref

pytestmark = pytest.mark.gpu

SHAPES = [
    # (logN nq qbits np pbits dnum), nlimbs, B
    ((13, 3, 50, 2, 60, 2), 3, 2),
    ((14, 5, 50, 2, 60, 3), 5, 3),    # digits 2, 2, 1; 4 tiles x odd slot counts
    ((14, 5, 50, 2, 60, 3), 4, 1),
    ((15, 4, 50, 3, 60, 2), 3, 2),
    ((13, 3, 60, 2, 60, 2), 3, 2),    # Harvey bodies throughout
    ((14, 3, 51, 2, 51, 2), 3, 2),    # uncorrected integer bodies throughout
    ((15, 3, 45, 2, 50, 3), 2, 2),    # double precision throughout, special primes too
]


@pytest.mark.parametrize("shape,nl,B", SHAPES)
def test_calls_on_the_smaller_two_pass_rings(shape, nl, B):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = make_params(*shape)
    rc, gc = ref.RefContext(p), gpu.Context(p)
    ids = list(range(nl))
    gs = [galois_element(k, p.logN) for k in (3, p.N // 4 + 1, 2 * B + 5)]
    ct, ct2 = (uniform_residues(70 + i, p.q[:nl], (B, 2), p.N) for i in range(2))
    ct[0, 0, 0, :], ct2[0, 1, nl - 1, :] = p.q[0] - 1, 0
    evks = [uniform_residues(80 + i, p.moduli, (p.dnum, 2), p.N) for i in range(3)]
    d_ct, d_ct2, d_evks = to_dev(ct), to_dev(ct2), [to_dev(k) for k in evks]
    ws, out = gc.workspace(gpu.OP_HROT, B, nl), torch.empty_like(d_ct)
    rots = [rc.hrot(ct, gs[i], evks[i]) for i in range(3)]
    gpu.ckks_hrot(gc, out, d_ct, B, nl, gs[0], d_evks[0], ws)
    assert_same(to_host(out), rots[0], "hrot")
    gpu.ckks_hrot_add(gc, out, d_ct, d_ct2, B, nl, gs[1], d_evks[1], ws)
    assert_same(to_host(out), rc.pointwise(ct2, rots[1], ids, "add"), "hrot_add")
    gpu.ckks_hrot_multi(gc, out, d_ct, B, nl, [gs[b % 3] for b in range(B)], [d_evks[b % 3] for b in range(B)], ws)
    assert_same(to_host(out), np.stack([rots[b % 3][b] for b in range(B)]), "hrot_multi")
    gpu.ckks_hmult_relin(gc, out, d_ct, d_ct2, B, nl, d_evks[2], ws)
    assert_same(to_host(out), rc.hmult_relin(ct, ct2, evks[2]), "hmult_relin")
    d3 = torch.empty((B, 3, nl, p.N), dtype=torch.int64, device="cuda")
    gpu.ckks_tensor_acc(gc, d3, d_ct, d_ct2, None, B, nl)
    gpu.ckks_relin(gc, out, d3, B, nl, d_evks[2], ws)
    assert_same(to_host(out), rc.hmult_relin(ct, ct2, evks[2]), "relin")
    rs = torch.empty((B, 2, nl - 1, p.N), dtype=torch.int64, device="cuda")
    gpu.ckks_rescale(gc, rs, d_ct, B, nl, gc.workspace(gpu.OP_RESCALE, B, nl))
    assert_same(to_host(rs), rc.rescale(ct), "rescale")
    # hoisted rotations: one at a time, and sharing passes over the digits in a larger workspace
    for extra in (0, 2 * B * 2 * (nl + len(p.p)) * p.N):
        big = torch.empty(ws.numel() + extra, dtype=torch.int64, device="cuda")
        h = torch.empty((3,) + tuple(out.shape), dtype=torch.int64, device="cuda")
        gpu.ckks_hrot_hoisted(gc, h, d_ct, B, nl, gs, d_evks, big)
        assert_same(to_host(h), np.stack(rots), "hrot_hoisted, %d words more" % extra)
    pt = uniform_residues(90, p.q[:nl], (2, 3), p.N)
    want = rc.pcmm_bsgs(ct, pt, 3, 2, 1, evks[:2], evks[2:])
    wsp = gc.workspace(gpu.OP_PCMM_BSGS, B, nl, 3)
    for call in (gpu.ckks_pcmm_bsgs, gpu.ckks_pcmm_bsgs_hoisted):
        call(gc, out, d_ct, B, nl, to_dev(pt), 3, 2, 1, d_evks[:2], d_evks[2:], wsp)
        assert_same(to_host(out), want, call.__name__)
    gc.close()
