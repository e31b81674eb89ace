"""Integer-class main limbs of a key switch on two-pass rings: finished in line by the kernel of the inner product, or, few of them with
many digits, from sums stored beside the special limbs'. Which way a call goes is read off its launches without a GPU."""
import pytest

import test_gpu_two_pass_rings as calls
from test_gpu_mixed_primes import mixed_params

IN_LINE, STORED, TENSOR = "inner8_kernelILi2ELb1E", "fwd_blocks_final_kernelILi2E", "tensor_kernel"
SHAPES = [
    # logN, sizes of the main primes, of the special primes, dnum; nlimbs, B; whether a rotation's sums are stored, a product's
    ((13, [60] + [50] * 4, [60], 5), 5, 4, True, True),
    ((13, [60, 60, 50, 50, 45, 50], [60, 60], 6), 4, 2, True, True),      # four digits at a lower level, two integer limbs
    ((13, [60] + [50] * 4, [60], 5), 3, 2, False, False),                 # three digits
    ((14, [60] * 6, [60], 6), 6, 4, True, True),                          # integers throughout
    ((13, [60] * 4, [60], 4), 4, 2, False, False),
    ((15, [60] + [50] * 3, [60], 4), 4, 16, True, False),                 # the most workgroups (512); too large a product
    ((15, [60] + [50] * 3, [60], 4), 4, 17, False, False),
]


@pytest.mark.parametrize("shape,nl,B,rotation,product", SHAPES)
def test_route(shape, nl, B, rotation, product):
    from launch_trace import trace
    steps = [name for what, _, name in trace(shape, {}, nl, B) if what == "launch"]
    halves = [i for i, k in enumerate(steps) if "inner8_kernelILi2ELb0E" in k]   # one launch of it a call, before the ones below
    assert len(halves) == 2
    ways = [[k for k in (IN_LINE, STORED) if any(k in s for s in part)] for part in (steps[halves[0]:halves[1]], steps[halves[1]:])]
    assert ways == [[STORED if rotation else IN_LINE], [STORED if product else IN_LINE]]
    assert any(TENSOR in s for s in steps) == product


@pytest.mark.gpu
@pytest.mark.parametrize("shape,nl,B,rotation,product", SHAPES)
def test_calls(shape, nl, B, rotation, product, monkeypatch):
    p = mixed_params(*shape)
    monkeypatch.setattr(calls, "make_params", lambda *s: p)
    calls.test_calls_on_the_smaller_two_pass_rings((), nl, B)
