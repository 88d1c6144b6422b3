"""Errors of the HIP runtime on the host side of the C ABI, on the CPU.

The library is loaded in a child process beside a stand-in for the runtime's
calls: device memory is host memory, kernels do nothing, asynchronous copies to
the host stay pending until their stream is waited for, and the n-th of them
can be made to fail.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
#include <string.h>
typedef int err;
typedef void* ptr;
static int pending, to_host, fail_at;
void fake_fail_at(int n) { fail_at = n; to_host = 0; }
int fake_pending(void) { return pending; }
err hipMemcpyAsync(ptr d, const void* s, size_t n, int kind, ptr st) {
  if (kind != 2) { memcpy(d, s, n); return 0; }
  if (++to_host == fail_at) return 1;
  ++pending;
  return 0;
}
err hipStreamSynchronize(ptr st) { pending = 0; return 0; }
err hipMemcpy(ptr d, const void* s, size_t n, int kind) { memcpy(d, s, n); return 0; }
err hipMemsetAsync(ptr d, int v, size_t n, ptr st) { memset(d, v, n); return 0; }
err hipStreamCreateWithFlags(ptr* st, unsigned f) { *st = (ptr)64; return 0; }
err hipStreamDestroy(ptr st) { return 0; }
err hipStreamWaitEvent(ptr st, ptr e, unsigned f) { return 0; }
err hipEventCreateWithFlags(ptr* e, unsigned f) { *e = (ptr)64; return 0; }
err hipEventDestroy(ptr e) { return 0; }
err hipEventRecord(ptr e, ptr st) { return 0; }
err hipEventQuery(ptr e) { return 0; }
err hipLaunchKernel(const void* f, ...) { return 0; }
err hipGetLastError(void) { return 0; }
const char* hipGetErrorString(err e) { return "stand-in error"; }
"""

PROGRAM = r"""
import ctypes as C, sys
import numpy as np
from paper_2512_09904_amd import cases, sph
fake = C.CDLL(sys.argv[1])
libc = C.CDLL(None)
libc.malloc.restype = C.c_void_p
libc.malloc.argtypes = [C.c_size_t]
libc.free.argtypes = [C.c_void_p]
L = sph.lib()
A = sph.Allocator(sph.ALLOC_FN(lambda n, s, u: libc.malloc(n)), sph.FREE_FN(lambda p, s, u: libc.free(p)), None)
c = cases.tank_c1(dp=5e-3)
P = sph.params_struct(c.params)
h = C.c_void_p()
assert L.sph_pool_create(C.c_size_t(1 << 40), 1, 0, C.byref(A), None, C.byref(h)) == 0
keep = [np.ascontiguousarray(a, np.float64) for a in (c.xf, c.vf, c.rhof, c.Tf, c.xs0, c.ns0)]
p = [a.ctypes.data_as(C.c_void_p) for a in keep]
body = np.ascontiguousarray(c.body, np.int32)
slot = C.c_int32()
assert L.sph_pool_admit(h, C.byref(P), len(c.bodies), sph.bodies_array(c.bodies), C.c_int64(c.nf), p[0], p[1], p[2],
                        p[3], None, C.c_int64(c.ns), p[4], p[5], body.ctypes.data_as(C.c_void_p), C.c_int64(5),
                        C.byref(slot)) == 0
out = [np.zeros(3 * c.nf), np.zeros(3 * c.nf), np.zeros(c.nf), np.zeros(c.nf)]
for n in range(5):
    fake.fake_fail_at(n)
    rc = L.sph_pool_get_fluid(h, slot, *[a.ctypes.data_as(C.c_void_p) for a in out])
    print(n, rc, fake.fake_pending(), flush=True)
L.sph_pool_destroy(h)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    src, so = d / "runtime.c", d / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.check_call(["gcc", "-w", "-shared", "-fPIC", "-O1", "-o", str(so), str(src)])
    return str(so)


def test_no_copy_into_the_callers_arrays_outlives_a_failed_read_out(runtime):
    """The fields are read out by up to four asynchronous copies.  When one of
    them fails the caller may free its arrays: none may still be in flight."""
    from paper_2512_09904_amd import sph
    env = dict(os.environ, LD_PRELOAD=runtime, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PROGRAM, runtime], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    got = [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
    assert got == [(0, sph.SPH_OK, 0)] + [(n, sph.SPH_ERR_HIP, 0) for n in (1, 2, 3, 4)]
