"""GPU parity of conversions of more than 8 sources: every number of groups of sources, short digits, groups of four targets that are
partly or wholly the digit's own limbs, both reductions, residues at the ends of their range, every kind of ring."""
import numpy as np
import pytest

import test_gpu_two_pass_rings as calls

pytestmark = pytest.mark.gpu

SHAPES = [
    # (logN nq qbits np pbits dnum), nlimbs, B
    ((13, 9, 50, 9, 60, 1), 9, 2),
    ((13, 24, 45, 13, 60, 2), 23, 1),     # 12 and 11 sources; own limbs in the middle of a group of targets
    ((14, 17, 60, 16, 60, 1), 17, 1),     # integers on both sides
    ((13, 23, 50, 23, 50, 1), 21, 1),     # double precision on both sides
    ((15, 36, 50, 30, 60, 1), 36, 1),
    ((13, 45, 55, 45, 60, 1), 45, 1),     # the most the library takes
    ((10, 20, 30, 10, 40, 2), 20, 3),     # one kernel per step
    ((11, 11, 60, 12, 60, 1), 10, 2),
    ((17, 10, 50, 9, 60, 1), 10, 1),
    ((16, 18, 52, 9, 60, 2), 17, 1),
]


@pytest.mark.parametrize("shape,nl,B", SHAPES)
def test_calls(shape, nl, B):
    calls.test_calls_on_the_smaller_two_pass_rings(shape, nl, B)


@pytest.mark.parametrize("shape", [(13, 36, 50, 36, 60, 1), (13, 45, 60, 45, 60, 1), (12, 24, 50, 24, 60, 1)])
def test_ends_of_the_range(shape):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import galois_element, make_params
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = make_params(*shape)
    rc, gc, nl, B = ref.RefContext(p), gpu.Context(p), len(p.q), 2
    top = np.array(p.moduli, dtype=np.uint64)[:, None]
    key = np.broadcast_to(top - np.uint64(1), (p.dnum, 2, len(p.moduli), p.N)).copy()
    ct = np.broadcast_to(top[:nl] // np.uint64(2), (B, 2, nl, p.N)).copy()
    ct[0, 1, ::2] += np.uint64(1)
    ct[1, 1, :, 1::2] = 0
    d_ct = to_dev(ct)
    out = torch.empty_like(d_ct)
    g = galois_element(5, p.logN)
    gpu.ckks_hrot(gc, out, d_ct, B, nl, g, to_dev(key), gc.workspace(gpu.OP_HROT, B, nl))
    assert_same(to_host(out), rc.hrot(ct, g, key), "hrot")
    gc.close()
