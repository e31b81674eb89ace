"""GPU parity of the few-launch key switch of the ring 2^12: every modulus class, both conversion reductions, more
sources than one chunk of a conversion, ragged digits and levels, more ciphertexts than one argument table; bit-exact."""
import numpy as np
import pytest

import test_gpu_two_pass_rings as calls
from ckks_inputs import galois_element, make_params, uniform_residues

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
