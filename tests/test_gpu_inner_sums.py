"""GPU parity of the diagonal matrix product's inner sums from 4 ciphertexts and 7 giant steps on, where they go through LDS if
that is estimated to be faster: tiles of 8 polynomials x 12 (integer limbs x 6) or x 8 giant steps, short last tiles, folds of
5 and 11 terms, both arithmetic kinds; bit-exact."""
import numpy as np
import pytest

from ckks_inputs import make_params, uniform_residues
from oracle import ref

pytestmark = pytest.mark.gpu

FP, INT, SMALL = (12, 3, 50, 2, 50, 2), (12, 3, 60, 2, 60, 2), (12, 3, 40, 2, 50, 2)
CASES = [
    # shape, B, n1, n2
    (FP, 4, 5, 12),      # one whole tile, one whole fold
    (FP, 5, 6, 9),       # a last tile of one ciphertext, a tile of 12 three quarters full, one term past a fold
    (FP, 4, 1, 7),       # one baby step: less than the copies in flight
    (FP, 4, 2, 8),
    (FP, 4, 11, 21),     # two tiles of 12 in one launch, the second short
    (FP, 4, 3, 27),      # giant steps beyond what the workspace holds at once: 24, then 3
    (SMALL, 7, 16, 10),
    (INT, 4, 11, 12),
    (INT, 5, 12, 9),     # register tiles
    (INT, 4, 1, 7),
    (INT, 4, 23, 8),
    (INT, 9, 2, 20),     # tiles of 6 and one of 8
]


@pytest.mark.parametrize("largest", [False, True])
@pytest.mark.parametrize("shape,B,n1,n2", CASES)
def test_inner_sums_through_lds(shape, B, n1, n2, largest):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = make_params(*shape)
    rc, gc, nl = ref.RefContext(p), gpu.Context(p), len(p.q)
    ct, pt = uniform_residues(1, p.q, (B, 2), p.N), uniform_residues(2, p.q, (n2, n1), p.N)
    if largest:       # the residues that the range arguments are made for
        top = np.array(p.q, dtype=np.uint64)[:, None] - np.uint64(1)
        ct[:], pt[:] = top, top
    baby = [uniform_residues(10 + i, p.moduli, (p.dnum, 2), p.N) for i in range(n1 - 1)]
    giant = [uniform_residues(50 + i, p.moduli, (p.dnum, 2), p.N) for i in range(n2 - 1)]
    ref.set_threads(8)
    want = rc.pcmm_bsgs(ct, pt, n1, n2, 1, baby, giant)
    ref.set_threads(1)
    d_ct, d_pt = to_dev(ct), to_dev(pt)
    args = (n1, n2, 1, [to_dev(k) for k in baby], [to_dev(k) for k in giant], gc.workspace(gpu.OP_PCMM_BSGS, B, nl, n1))
    out = torch.empty_like(d_ct)
    gpu.ckks_pcmm_bsgs(gc, out, d_ct, B, nl, d_pt, *args)
    assert_same(to_host(out), want, "inner sums")
    # rows that 16-byte copies cannot start at take the kernels without LDS: the same bits
    shifted = torch.empty(d_pt.numel() + 1, dtype=torch.int64, device="cuda")[1:].view_as(d_pt)
    shifted.copy_(d_pt)
    out.zero_()
    gpu.ckks_pcmm_bsgs(gc, out, d_ct, B, nl, shifted, *args)
    assert_same(to_host(out), want, "inner sums, plaintexts on an odd word")
    gc.close()


def _ran(gpu, gc, call):
    gpu.ckks_prof_reset(gc)
    gpu.ckks_prof_enable(gc, True)
    call()
    gpu.ckks_prof_enable(gc, False)
    return {k for k in gpu.ckks_prof_collect(gc) if k.startswith("pmacc")}


@pytest.mark.parametrize("shape,kind", [(FP, "pmacc_fp"), (INT, "pmacc_int")])
def test_profile_names_the_kernel_that_ran(shape, kind):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import to_dev
    p = make_params(*shape)
    gc, nl, B, n1, n2 = gpu.Context(p), len(p.q), 4, 3, 8
    d_ct, d_pt = to_dev(uniform_residues(1, p.q, (B, 2), p.N)), to_dev(uniform_residues(2, p.q, (n2, n1), p.N))
    key = to_dev(uniform_residues(3, p.moduli, (p.dnum, 2), p.N))
    shifted = torch.empty(d_pt.numel() + 1, dtype=torch.int64, device="cuda")[1:].view_as(d_pt)
    shifted.copy_(d_pt)
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_PCMM_BSGS, B, nl, n1)
    for pt, ran, other in ((d_pt, "_staged_kernel", "_kernel"), (shifted, "_kernel", "_staged_kernel")):
        times = _ran(gpu, gc, lambda: gpu.ckks_pcmm_bsgs(gc, out, d_ct, B, nl, pt, n1, n2, 1, [key] * (n1 - 1), [key] * (n2 - 1), ws))
        assert kind + ran in times and kind + other not in times, times
    gc.close()


@pytest.mark.parametrize("shape,B,n1,n2,staged", [
    (FP, 8, 1, 18, False),      # three whole register tiles in one launch
    (FP, 8, 1, 24, False),
    (FP, 4, 8, 8, True),
    (FP, 5, 8, 13, True),       # two tiles of 8
    (FP, 4, 16, 23, True),      # two tiles of 12, the last one short
    (FP, 3, 16, 8, False),
    (FP, 4, 16, 6, False),
    (INT, 5, 3, 18, False),     # six register tiles of 3
    (INT, 5, 8, 9, False),
    (INT, 5, 5, 7, True),
    (INT, 4, 4, 13, True),      # three tiles of 6, one giant step in the last
    (INT, 4, 16, 22, True),     # four tiles of 6, the last one short
])
def test_kernels_of_the_inner_sums(shape, B, n1, n2, staged):
    """Staged through LDS only where that was measured faster than whole register tiles; the bits are the oracle's."""
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p = make_params(*shape)
    rc, gc, nl, some = ref.RefContext(p), gpu.Context(p), len(p.q), [0, B - 1]
    ct, pt = uniform_residues(1, p.q, (B, 2), p.N), uniform_residues(2, p.q, (n2, n1), p.N)
    key = uniform_residues(3, p.moduli, (p.dnum, 2), p.N)
    d_ct, d_pt, d_key = to_dev(ct), to_dev(pt), to_dev(key)
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_PCMM_BSGS, B, nl, n1)
    ran = _ran(gpu, gc, lambda: gpu.ckks_pcmm_bsgs(gc, out, d_ct, B, nl, d_pt, n1, n2, 1, [d_key] * (n1 - 1), [d_key] * (n2 - 1), ws))
    kind = "pmacc_fp" if shape is FP else "pmacc_int"
    assert ran == {kind + ("_staged_kernel" if staged else "_kernel")}
    ref.set_threads(8)
    want = rc.pcmm_bsgs(ct[some], pt, n1, n2, 1, [key] * (n1 - 1), [key] * (n2 - 1))
    ref.set_threads(1)
    assert_same(to_host(out)[some], want, "inner sums")
    gc.close()


@pytest.mark.parametrize("B,n1,n2", [
    (4, 3, 7),       # tiles of 8 for both kinds of limbs
    (4, 3, 11),      # one tile of 12, two of 6
    (5, 12, 11),     # past a fold of either kind
])
def test_inner_sums_through_lds_in_the_extended_basis(B, n1, n2):
    """Main limbs below the top level and special ones after them (a limb's modulus is not its index), both arithmetic kinds
    writing to the same sums."""
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    p, nl = make_params(16, 4, 50, 2, 60, 2), 3
    rc, gc, some = ref.RefContext(p), gpu.Context(p), [0, B - 1]
    ct, pt = uniform_residues(1, p.q[:nl], (B, 2), p.N), uniform_residues(2, list(p.q[:nl]) + list(p.p), (n2, n1), p.N)
    keys = [uniform_residues(3 + i, p.moduli, (p.dnum, 2), p.N) for i in range(3)]
    baby, giant = [keys[i % 3] for i in range(n1 - 1)], [keys[(i + 1) % 3] for i in range(n2 - 1)]
    d_ct, d_pt, d_keys = to_dev(ct), to_dev(pt), [to_dev(k) for k in keys]
    d_baby, d_giant = [d_keys[i % 3] for i in range(n1 - 1)], [d_keys[(i + 1) % 3] for i in range(n2 - 1)]
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_PCMM_BSGS_DH, B, nl, n1)
    ran = _ran(gpu, gc, lambda: gpu.ckks_pcmm_bsgs_double_hoisted(gc, out, d_ct, B, nl, d_pt, n1, n2, 1, d_baby, d_giant, ws))
    assert ran == {"pmacc_fp_staged_kernel", "pmacc_int_staged_kernel"}
    ref.set_threads(8)
    want = rc.pcmm_bsgs_double_hoisted(ct[some], pt, n1, n2, 1, baby, giant)
    ref.set_threads(1)
    assert_same(to_host(out)[some], want, "extended basis")
    gc.close()


@pytest.mark.parametrize("logN,B,n1,n2", [(13, 5, 6, 11), (12, 4, 12, 8)])
def test_inner_sums_through_lds_on_mixed_primes(logN, B, n1, n2):
    import torch
    import paper_2604_03425_amd as gpu
    from gpu_util import assert_same, to_dev, to_host
    from test_gpu_mixed_primes import mixed_params
    p, nl = mixed_params(logN, [60, 50, 50, 60], [60, 60], 2), 3
    rc, gc = ref.RefContext(p), gpu.Context(p)
    ct, pt = uniform_residues(1, p.q[:nl], (B, 2), p.N), uniform_residues(2, p.q[:nl], (n2, n1), p.N)
    baby = [uniform_residues(10 + i, p.moduli, (p.dnum, 2), p.N) for i in range(n1 - 1)]
    giant = [uniform_residues(50 + i, p.moduli, (p.dnum, 2), p.N) for i in range(n2 - 1)]
    d_ct, d_pt, d_baby, d_giant = to_dev(ct), to_dev(pt), [to_dev(k) for k in baby], [to_dev(k) for k in giant]
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_PCMM_BSGS, B, nl, n1)
    ran = _ran(gpu, gc, lambda: gpu.ckks_pcmm_bsgs(gc, out, d_ct, B, nl, d_pt, n1, n2, 1, d_baby, d_giant, ws))
    assert ran == {"pmacc_fp_staged_kernel", "pmacc_int_staged_kernel"}
    ref.set_threads(8)
    want = rc.pcmm_bsgs(ct, pt, n1, n2, 1, baby, giant)
    ref.set_threads(1)
    assert_same(to_host(out), want, "mixed primes")
    gc.close()
