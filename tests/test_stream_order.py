"""Order of a key switch's kernels on its two streams (knob 4 = 0), read off the launches: the library runs on a stand-in for the HIP
runtime that writes down every launch, event record and wait and executes nothing, so this needs no GPU."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <map>
struct dim3 { unsigned x, y, z; };
static std::map<const void*, const char*>& kernels() { static std::map<const void*, const char*> k; return k; }
static intptr_t handles = 1;
static struct { dim3 grid, block; size_t shared; void* stream; } config;
static char symbol[64];
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { config = {g, b, s, st}; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = config.grid, *b = config.block, *s = config.shared, *st = config.stream; return 0; }
int hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, void* st) { printf("launch %ld %s\n", (long)(intptr_t)st, kernels()[f]); return 0; }
int hipEventRecord(void* e, void* st) { printf("record %ld %ld\n", (long)(intptr_t)st, (long)(intptr_t)e); return 0; }
int hipStreamWaitEvent(void* st, void* e, unsigned) { printf("wait %ld %ld\n", (long)(intptr_t)st, (long)(intptr_t)e); return 0; }
int hipStreamCreateWithFlags(void** st, unsigned) { *st = (void*)++handles; return 0; }
int hipEventCreate(void** e) { *e = (void*)++handles; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)++handles; return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, void*) { return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = symbol; return 0; }
const char* hipGetErrorString(int) { return ""; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) { *t = 0; return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
}
"""

CALLS = r"""
import ctypes as C, json, sys
from ckks_inputs.params import CkksParams, find_ntt_primes, find_psi
logN, q_bits, p_bits, dnum, knobs = json.loads(sys.argv[2])
primes = []
for bits in q_bits + p_bits:
    primes += find_ntt_primes(bits, 1, logN, exclude=set(primes))
nq = len(q_bits)
lib = C.CDLL(sys.argv[1])
lib.ckks_workspace_bytes.restype = C.c_size_t
lib.ckks_last_error.restype = C.c_char_p
def array(v): return (C.c_uint64 * len(v))(*v)
def check(rc):
    if rc: sys.exit(lib.ckks_last_error().decode())
ctx = C.c_void_p()
check(lib.ckks_ctx_create(C.byref(ctx), logN, array(primes[:nq]), nq, array(primes[nq:]), len(p_bits), dnum,
                          array([find_psi(m, logN) for m in primes]), 0))
for k, v in knobs:
    check(lib.ckks_tune_set(ctx, k, v))
a, b, out, key, ws, st = (C.c_void_p(n << 40) for n in (1, 2, 3, 4, 5, 6))
n = C.c_size_t(lib.ckks_workspace_bytes(ctx, 3, 2, nq, 0))
check(lib.ckks_hrot(ctx, out, a, 2, nq, 5, key, ws, n, st))
check(lib.ckks_hmult_relin(ctx, out, a, b, 2, nq, key, ws, n, st))
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    (d / "hip.cpp").write_text(RUNTIME)
    (d / "hip.map").write_text("hip_4.2 { global: hip*; __hip*; local: *; };\n")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-o", str(d / "libamdhip64.so.7"), str(d / "hip.cpp"),
                    "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script," + str(d / "hip.map")], check=True)
    return d


def _trace(runtime, shape, knobs):
    import json
    import paper_2604_03425_amd as pkg
    env = dict(os.environ, LD_LIBRARY_PATH=str(runtime), PYTHONPATH=ROOT)
    res = subprocess.run([sys.executable, "-c", CALLS, pkg.library_path(), json.dumps(list(shape) + [sorted(knobs.items())])],
                         env=env, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stderr
    return [line.split() for line in res.stdout.splitlines()]


def _before(trace):
    """Per launch (name, stream): the set of earlier launches that it is ordered after."""
    seen, events, out = {}, {}, []
    for what, stream, arg in trace:
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
def test_second_stream_is_joined_before_its_digits_are_read(runtime, shape, knobs):
    launches = _before(_trace(runtime, shape, knobs))
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
