"""GPU parity of key switches whose special limbs leave the inner product through their inverse block pass: special primes of every
class, alone and mixed, sums at the ends of their range."""
import numpy as np
import pytest

from ckks_inputs import galois_element
from test_gpu_mixed_primes import mixed_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,q_bits,p_bits,dnum,B", [
    (13, [50, 50, 50], [52, 52], 3, 2),
    (14, [50, 50, 50, 50], [60, 51], 2, 1),
    (13, [60, 60], [60], 2, 3),
    (15, [50, 50], [50, 60, 52], 1, 1),   # a double-precision special prime beside both integer classes
    (16, [52, 52], [60], 2, 1),
])
def test_special_limbs(logN, q_bits, p_bits, dnum, B):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(logN, q_bits, p_bits, dnum)
    rc, gc, nl = ref.RefContext(p), gpu.Context(p), len(p.q)
    top = np.array(p.moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    key = np.broadcast_to(top, (p.dnum, 2, len(p.moduli), p.N)).copy()
    key[:, 1, :, ::3] = 0
    ct = np.broadcast_to(top[:nl], (B, 2, nl, p.N)).copy()
    ct[0, 1, :, 1::2] = 0
    g = galois_element(3, p.logN)
    d_ct = to_dev(ct)
    out = torch.empty_like(d_ct)
    gpu.ckks_hrot(gc, out, d_ct, B, nl, g, to_dev(key), gc.workspace(gpu.OP_HROT, B, nl))
    assert_same(to_host(out), rc.hrot(ct, g, key), "hrot")
    gc.close()
