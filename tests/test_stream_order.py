"""Order of a key switch's kernels on its two streams (knob 4 = 0), read off the launches."""
import pytest

from launch_trace import trace


def _before(steps):
    """Per launch (name, stream): the set of earlier launches that it is ordered after."""
    seen, events, out = {}, {}, []
    for what, stream, arg in steps:
        s = seen.setdefault(stream, set())
        if what == "launch":
            out.append((arg, stream, frozenset(s)))
            s.add(len(out) - 1)
        elif what == "record":
            events[arg] = frozenset(s)
        else:
            s |= events.get(arg, frozenset())
    return out


SHAPES = [
    # logN, sizes of the main primes, of the special primes, dnum
    (13, [50] * 4, [60] * 2, 2),
    (13, [50] * 9, [60] * 9, 1),              # more sources than the fused conversion takes
    (14, [60, 50, 50, 50], [60] * 2, 2),      # both kinds among the main primes
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("knobs", [{4: 0}, {2: 2, 4: 0}, {3: 1, 4: 0}, {2: 2, 3: 1, 4: 0}])
def test_second_stream_is_joined_before_its_digits_are_read(shape, knobs):
    launches = _before(trace(shape, knobs))
    main = launches[0][1]
    side = [i for i, (_, stream, _) in enumerate(launches) if stream != main]
    fused = shape[1] == [50] * 4 and 2 not in knobs   # conversion and row pass in one kernel: nothing to run beside it
    assert len(side) == (0 if fused else 2)           # one row pass a call
    readers = 0
    for i, (name, stream, after) in enumerate(launches):
        assert stream == main or "fwd_rows_kernelILi0E" in name
        # what reads (or transforms in place) the converted digits of double-precision limbs
        if any(k in name for k in ("fwd_blocks_kernelILi0E", "inner16_fp_kernel", "blocks_inner_c_kernel")):
            readers += 1
            assert after >= {k for k in side if k < i}, (name, "is not ordered after the row pass on the second stream")
    assert readers >= 2
    assert launches[-1][2] >= set(side)   # and the caller's stream goes on only after it
