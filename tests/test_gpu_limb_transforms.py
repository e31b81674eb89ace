"""GPU parity of the transforms that hold a limb per workgroup (N = 2^10 .. 2^14): every length of the last round, the three
modulus classes side by side, residues at the ends of their range, data aligned to one word only."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN", [10, 11, 12, 13, 14])
@pytest.mark.parametrize("q_bits,p_bits", [(50, 60), (51, 40), (52, 60)])
def test_whole_transforms(logN, q_bits, p_bits):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import make_params, uniform_residues
    from gpu_util import assert_same, to_host
    from oracle import ref
    p = make_params(logN, 2, q_bits, 1, p_bits, 1)
    rc, gc = ref.RefContext(p), gpu.Context(p)
    ids, B = [2, 0, 1], 4
    mods = [p.moduli[i] for i in ids]
    x = uniform_residues(7 * logN + q_bits, mods, (B,), p.N)
    for i, m in enumerate(mods):
        x[0, i, :] = m - 1
        x[1, i, ::2], x[1, i, 1::2] = 0, m - 1
        x[2, i, : p.N // 2], x[2, i, p.N // 2:] = m - 1, 0
    for offset in (0, 1):
        for fn, want in ((gpu.ckks_ntt, rc.ntt(x, ids)), (gpu.ckks_intt, rc.intt(x, ids))):
            buf = torch.zeros(x.size + 2, dtype=torch.int64, device="cuda")
            d = buf[offset:offset + x.size].view(x.shape)
            d.copy_(torch.from_numpy(x.view(np.int64)))
            fn(gc, d, B, ids)
            assert_same(to_host(d), want, "%s at word %d" % (fn.__name__, offset))
            assert int(buf[:offset].sum()) == 0 and int(buf[offset + x.size:].sum()) == 0
    gc.close()
