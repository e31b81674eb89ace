"""The launches of a few calls, without a GPU: the library runs on a stand-in for the HIP runtime that writes down every launch, event
record and wait and executes nothing."""
import json
import os
import subprocess
import sys
import tempfile

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
logN, q_bits, p_bits, dnum, knobs, nl, B, calls = json.loads(sys.argv[2])
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
nl = nl or nq
n = C.c_size_t(lib.ckks_workspace_bytes(ctx, 3, B, nl, 0))
ids = (C.c_uint32 * nl)(*range(nl))
for call in calls:
    if call == "hrot": check(lib.ckks_hrot(ctx, out, a, B, nl, 5, key, ws, n, st))
    if call == "hmult": check(lib.ckks_hmult_relin(ctx, out, a, b, B, nl, key, ws, n, st))
    if call == "ntt": check(lib.ckks_ntt(ctx, a, B, ids, nl, st))
    if call == "intt": check(lib.ckks_intt(ctx, a, B, ids, nl, st))
"""

_folder = None


def _runtime():
    """The folder of the stand-in, built once."""
    global _folder
    if _folder is None:
        _folder = tempfile.TemporaryDirectory()
        src, names = os.path.join(_folder.name, "hip.cpp"), os.path.join(_folder.name, "hip.map")
        open(src, "w").write(RUNTIME)
        open(names, "w").write("hip_4.2 { global: hip*; __hip*; local: *; };\n")
        subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-o", os.path.join(_folder.name, "libamdhip64.so.7"), src,
                        "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script," + names], check=True)
    return _folder.name


def trace(shape, knobs, nl=0, B=2, calls=("hrot", "hmult")):
    """("launch", stream, kernel), ("record" or "wait", stream, event) of `calls` on B ciphertexts (transforms: polynomials)
    of nl limbs (0: all). shape: logN, sizes of the main primes, of the special primes, digits."""
    import paper_2604_03425_amd as pkg
    env = dict(os.environ, LD_LIBRARY_PATH=_runtime(), PYTHONPATH=ROOT)
    res = subprocess.run([sys.executable, "-c", CALLS, pkg.library_path(),
                          json.dumps(list(shape) + [sorted(knobs.items()), nl, B, calls])], env=env,
                         stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stderr
    return [line.split() for line in res.stdout.splitlines()]
