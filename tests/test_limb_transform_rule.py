"""Ring 2^14: whole transforms hold a limb per workgroup where that fills the chip, or where the limbs are of two arithmetic kinds, and
take the two-pass kernels elsewhere. The form is read off the launches without a GPU; on it both are compared with the oracle."""
import pytest

from test_gpu_mixed_primes import mixed_params

CASES = [
    # sizes of the primes, polynomials, whether a limb per workgroup
    ([50], 1, False), ([50], 128, False), ([50], 129, True), ([50, 50, 50], 85, True), ([50], 257, False),
    ([50, 50], 192, False), ([50, 50], 193, True), ([50], 513, False), ([50], 641, True),
    ([60], 2, False), ([60], 129, True), ([60], 385, True), ([51], 641, False), ([60, 60], 353, True), ([51], 128, False),
    ([50, 60], 1, True), ([51, 60], 1, True), ([50, 50, 51], 100, True), ([50], 2049, True),
]


@pytest.mark.parametrize("bits,npoly,whole", CASES)
def test_route(bits, npoly, whole):
    from launch_trace import trace
    for call in ("ntt", "intt"):
        kernels = [name for what, _, name in trace((14, bits, [40], 1), {}, len(bits), npoly, [call]) if what == "launch"]
        assert len(kernels) == (1 if whole else 2) and all(("ntt_limb_kernel" in k) == whole for k in kernels), kernels


DIRECTIONS = [
    # size of the primes, limbs, whether a limb per workgroup: forward, inverse
    (50, 1024, True, True), (50, 1280, True, False), (50, 2048, True, False), (50, 2049, True, True),
    (51, 512, True, True), (51, 768, True, False), (51, 1024, True, False), (51, 1280, False, False), (51, 2176, True, False),
    (51, 2177, True, True), (60, 641, True, False), (60, 768, True, True), (60, 1024, True, False), (60, 2048, True, False), (60, 2305, True, True),
]


@pytest.mark.parametrize("bits,limbs,forward,inverse", DIRECTIONS)
def test_route_of_each_direction(bits, limbs, forward, inverse):
    from launch_trace import trace
    for call, whole in (("ntt", forward), ("intt", inverse)):
        kernels = [name for what, _, name in trace((14, [bits], [40], 1), {}, 1, limbs, [call]) if what == "launch"]
        assert len(kernels) == (1 if whole else 2) and all(("ntt_limb_kernel" in k) == whole for k in kernels), kernels


def test_other_rings_have_one_form():
    from launch_trace import trace
    for logN, kernel in ((10, "ntt_limb_kernelILi10E"), (13, "ntt_limb_kernelILi13E"), (15, "ntt16_"), (17, "ntt_pass_kernel")):
        steps = trace((logN, [50], [60], 1), {}, 1, 1, ["ntt", "intt"])
        assert all(kernel in name for what, _, name in steps if what == "launch")


@pytest.mark.gpu
@pytest.mark.parametrize("bits,npoly", [c[:2] for c in CASES if c[1] <= 257] + [([51], 1024)])
def test_parity(bits, npoly):
    import torch
    import paper_2604_03425_amd as gpu
    from ckks_inputs import uniform_residues
    from gpu_util import assert_same, to_dev, to_host
    from oracle import ref
    p = mixed_params(14, bits, [40], 1)
    rc, gc, ids = ref.RefContext(p), gpu.Context(p), list(range(len(bits)))
    x = uniform_residues(npoly, p.q, (npoly,), p.N)
    x[0] = [[m - 1] for m in p.q]
    for fn, want in ((gpu.ckks_ntt, rc.ntt), (gpu.ckks_intt, rc.intt)):
        d = to_dev(x)
        fn(gc, d, npoly, ids)
        assert_same(to_host(d), want(x, ids), fn.__name__)
    gc.close()
