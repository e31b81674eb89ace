"""Which conversion kernels a call takes: read off the launches without a GPU, and on it the same calls against the oracle, so that
every form of the conversions that are kernels of their own is known to be compared."""
import pytest

from test_gpu_mixed_primes import mixed_params

FUSED = "conv_rows_kernel"


def _own(kernel, sources, prescaled, narrow):
    return "%s_kernelILi%dELb%dELb%dE" % (kernel, sources, prescaled, narrow)


S4, S8 = (13, [50] * 4, [60] * 3, 1), (13, [50] * 8, [60] * 8, 1)
LARGE = (16, [50] * 5, [60] * 3, 2)
STEPS4, STEPS8 = (11, [50] * 4, [60] * 3, 1), (11, [50] * 8, [60] * 8, 1)
ROUTES = [
    # (logN, sizes of the main primes, of the special primes, dnum), knobs, ModUp's kernel, ModDown's
    (S4, {}, FUSED, FUSED),
    (S4, {5: 1}, FUSED, FUSED),      # the fused conversion knows one form
    (S4, {2: 2}, _own("modup", 4, 1, 1), _own("moddown", 4, 1, 1)),
    (S4, {2: 2, 5: 1}, _own("modup", 4, 1, 0), _own("moddown", 4, 1, 0)),
    (S4, {2: 2, 4: 0, 5: 1}, _own("modup", 4, 1, 0), _own("moddown", 4, 1, 0)),
    (S8, {2: 2}, _own("modup", 8, 1, 1), _own("moddown", 8, 1, 1)),
    (S8, {2: 2, 5: 1}, _own("modup", 8, 1, 0), _own("moddown", 8, 1, 0)),
    # 8 sources up to 60 bits beside one of the other arithmetic kind: the general form without any knob
    ((13, [60] * 7 + [50], [60] * 7 + [50], 1), {}, _own("modup", 8, 1, 0), _own("moddown", 8, 1, 0)),
    (LARGE, {2: 2, 5: 1}, _own("modup", 4, 1, 0), _own("moddown", 4, 1, 0)),
    (LARGE, {2: 2, 4: 0, 5: 1}, _own("modup", 4, 1, 0), _own("moddown", 4, 1, 0)),
    (STEPS4, {}, _own("modup", 4, 0, 1), _own("moddown", 4, 0, 1)),
    (STEPS4, {5: 1}, _own("modup", 4, 0, 0), _own("moddown", 4, 0, 0)),
    (STEPS8, {}, _own("modup", 8, 0, 1), _own("moddown", 8, 0, 1)),
    (STEPS8, {5: 1}, _own("modup", 8, 0, 0), _own("moddown", 8, 0, 0)),
]


@pytest.mark.parametrize("shape,knobs,up,down", ROUTES)
def test_route(shape, knobs, up, down):
    from launch_trace import trace
    kernels = {name for what, _, name in trace(shape, knobs) if what == "launch"}
    assert any(up in k for k in kernels) and any(down in k for k in kernels), kernels
    conversions = {k for k in kernels if any(c in k for c in (FUSED, "modup_kernel", "moddown_kernel", "conv_wide", "bconv_rows"))}
    assert all(up in k or down in k for k in conversions), conversions


def test_every_form_is_taken():
    assert {r for _, _, up, down in ROUTES for r in (up, down)} >= {
        _own(k, n, p, w) for k in ("modup", "moddown") for n in (4, 8) for p in (0, 1) for w in (0, 1)}


@pytest.mark.gpu
@pytest.mark.parametrize("shape,knobs,up,down", ROUTES)
def test_parity(shape, knobs, up, down):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import galois_element, uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(*shape)
    rc, gc, nl, B = ref.RefContext(p), gpu.Context(p), len(p.q), 2
    for k, v in knobs.items():
        gpu.ckks_tune_set(gc, k, v)
    ct, ct2 = (uniform_residues(60 + i, p.q, (B, 2), p.N) for i in range(2))
    ct[0] = [[[m - 1] for m in p.q]] * 2
    evk, g = uniform_residues(62, p.moduli, (p.dnum, 2), p.N), galois_element(9, p.logN)
    d_ct, d_ct2, d_evk = to_dev(ct), to_dev(ct2), to_dev(evk)
    out, ws = torch.empty_like(d_ct), gc.workspace(gpu.OP_HROT, B, nl)
    gpu.ckks_hrot(gc, out, d_ct, B, nl, g, d_evk, ws)
    assert_same(to_host(out), rc.hrot(ct, g, evk), "hrot")
    gpu.ckks_hmult_relin(gc, out, d_ct, d_ct2, B, nl, d_evk, ws)
    assert_same(to_host(out), rc.hmult_relin(ct, ct2, evk), "hmult_relin")
    low = torch.empty((B, 2, nl - 1, p.N), dtype=torch.int64, device=d_ct.device)
    gpu.ckks_rescale(gc, low, d_ct, B, nl, gc.workspace(gpu.OP_RESCALE, B, nl))
    assert_same(to_host(low), rc.rescale(ct), "rescale")
    gc.close()


@pytest.mark.gpu
def test_matrix_products_in_the_general_form():
    """Both schedules of a matrix product with the conversions as kernels of their own in the general form."""
    import numpy as np
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(*LARGE)
    rc, gc, nl, B, n1, n2 = ref.RefContext(p), gpu.Context(p), len(p.q), 2, 3, 2
    gpu.ckks_tune_set(gc, 2, 2)
    gpu.ckks_tune_set(gc, 5, 1)
    ct, pte = uniform_residues(1, p.q, (B, 2), p.N), uniform_residues(2, list(p.q) + list(p.p), (n2, n1), p.N)
    pt = np.ascontiguousarray(pte[:, :, :nl])
    bk, gk = ([uniform_residues(s + i, p.moduli, (p.dnum, 2), p.N) for i in range(n - 1)] for s, n in ((10, n1), (20, n2)))
    d_ct, dbk, dgk = to_dev(ct), [to_dev(k) for k in bk], [to_dev(k) for k in gk]
    out = torch.empty_like(d_ct)
    gpu.ckks_pcmm_bsgs_double_hoisted(gc, out, d_ct, B, nl, to_dev(pte), n1, n2, 1, dbk, dgk, gc.workspace(gpu.OP_PCMM_BSGS_DH, B, nl, n1))
    assert_same(to_host(out), rc.pcmm_bsgs_double_hoisted(ct, pte, n1, n2, 1, bk, gk), "extended-basis schedule")
    gpu.ckks_pcmm_bsgs_hoisted(gc, out, d_ct, B, nl, to_dev(pt), n1, n2, 1, dbk, dgk, gc.workspace(gpu.OP_PCMM_BSGS, B, nl, n1))
    assert_same(to_host(out), rc.pcmm_bsgs(ct, pt, n1, n2, 1, bk, gk), "hoisted schedule")
    gc.close()
