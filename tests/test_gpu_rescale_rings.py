"""GPU parity of the rescale on two-pass rings: dropped primes of every class against remaining primes of every class, residues at the
ends of their range and around half the dropped prime, where the centred representative changes sign."""
import numpy as np
import pytest

from test_gpu_mixed_primes import mixed_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,q_bits,B", [
    (13, [50, 50], 1),
    (13, [60, 52, 50, 51], 3),
    (14, [50, 60], 2),
    (14, [52, 50, 60, 50, 40], 1),
    (15, [50, 45, 60], 2),
    (16, [60, 50, 52], 1),
])
def test_rescale(logN, q_bits, B):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(logN, q_bits, [60], 1)
    rc, gc = ref.RefContext(p), gpu.Context(p)
    rng = np.random.default_rng(5)
    for nl in range(2, len(p.q) + 1):
        q = np.array(p.q[:nl], dtype=np.uint64)[:, None]
        ct = np.empty((B, 2, nl, p.N), dtype=np.uint64)
        for i in range(nl):
            ct[:, :, i] = rng.integers(0, p.q[i], (B, 2, p.N), dtype=np.uint64)
        ct[0, 0] = q - np.uint64(1)
        # a constant polynomial's transform is that constant: the dropped limb holds (q - 1) / 2 and (q + 1) / 2 at coefficient 0
        ct[0, 1, -1] = (q[-1, 0] - np.uint64(1)) // np.uint64(2)
        ct[B - 1, 1, -1] = (q[-1, 0] + np.uint64(1)) // np.uint64(2)
        d_ct = to_dev(ct)
        out = torch.empty((B, 2, nl - 1, p.N), dtype=torch.int64, device=d_ct.device)
        gpu.ckks_rescale(gc, out, d_ct, B, nl, gc.workspace(gpu.OP_RESCALE, B, nl))
        assert_same(to_host(out), rc.rescale(ct), "rescale of %d limbs" % nl)
    gc.close()
