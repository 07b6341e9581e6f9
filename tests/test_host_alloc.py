"""Device memory of the evaluation plans, on the CPU: a stand-in for the HIP runtime's
memory and launch calls (host memory, launches that do nothing) counts what the
library allocates and refuses what a test asks it to.  Each scenario runs in a
process of its own, in which the stand-in is loaded before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
long live = 0, calls = 0, launches = 0, fail_at = 0, max_bytes = -1;
int capturing = 0;
int hipMalloc(void** p, size_t n) {
  ++calls;
  *p = NULL;
  if (calls == fail_at || (max_bytes >= 0 && (long)n > max_bytes)) return 2; /* out of memory */
  char* b = calloc(1, n + 64);
  if (!b) return 2;
  *(size_t*)b = n;
  live += n;
  *p = b + 64;
  return 0;
}
int hipFree(void* p) {
  if (!p) return 0;
  live -= *(size_t*)((char*)p - 64);
  free((char*)p - 64);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int k) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { memcpy(d, s, n); return 0; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void* s) { return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* l, void** s) {
  *g = *b = (dim3_t){1, 1, 1};
  *l = 0;
  *s = NULL;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t l, void* s) { ++launches; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamIsCapturing(void* s, int* st) { *st = capturing; return 0; }
"""

PRELUDE = """
import ctypes, sys
import numpy as np
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
var = lambda n: ctypes.c_long.in_dll(stub, n)
from paper_2504_12004_amd import sbv

def handle(joint, count, own=1):
    # `count` blocks of `own` points each on the `joint - own` points before them
    lead = joint - own
    sizes = [1] * lead + [own] * count
    bp = np.r_[0, np.cumsum(sizes)]
    n = int(bp[-1])
    idx = [np.arange(bp[r] - (lead if r >= lead else 0), bp[r]) for r in range(len(sizes))]
    X = np.random.default_rng(0).random((n, 2))
    return sbv.sbv_blocks_import(X, np.zeros(n), bp, np.arange(n), np.r_[0, np.cumsum([len(i) for i in idx])],
                                 np.concatenate(idx))

theta = np.zeros(4)
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    d = tmp_path_factory.mktemp("stub")
    (d / "stub.c").write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(d / "stub.so"), str(d / "stub.c")], check=True)
    return str(d / "stub.so")


def _run(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), stub], cwd=ROOT, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_gradient_after_running_out_of_memory(stub):
    """Whichever allocation of the first gradient call fails, the next call has the
    buffers that an undisturbed one has."""
    _run(stub, """
    def grad(h, fail):
        before = var("calls").value
        var("fail_at").value = before + fail if fail else 0
        st = sbv.SBV_OK
        try:
            sbv.sbv_loglik_grad(h, theta, 5)
        except sbv.SBVError as e:
            st = e.status
        var("fail_at").value = 0
        return st, var("calls").value - before

    def fresh():
        h = handle(100, 20)
        sbv.sbv_loglik(h, theta, 5, sbv.SBV_FP32)  # the plan
        return h

    h = fresh()
    st, count = grad(h, 0)
    whole = var("live").value
    assert st == 0 and count >= 4, (st, count)
    h.free()
    for i in range(1, count + 1):
        h = fresh()
        assert grad(h, i)[0] == sbv.SBV_E_NOMEM
        assert grad(h, 0)[0] == 0
        assert var("live").value == whole, (i, var("live").value, whole)
        assert grad(h, 0) == (0, 0)
        h.free()
    assert var("live").value == 0
    """)


def test_simulation_after_running_out_of_memory(stub):
    """Likewise the first simulation's work lists and buffers."""
    _run(stub, """
    def sample(h, fail):
        before = var("calls").value
        var("fail_at").value = before + fail if fail else 0
        st = sbv.SBV_OK
        try:
            sbv.sbv_sample(h, theta, 5, np.zeros(119))
        except sbv.SBVError as e:
            st = e.status
        var("fail_at").value = 0
        return st, var("calls").value - before

    h = handle(100, 20)
    st, count = sample(h, 0)
    whole = var("live").value
    assert st == 0 and count >= 8, (st, count)
    h.free()
    for i in range(1, count + 1):
        h = handle(100, 20)
        assert sample(h, i)[0] == sbv.SBV_E_NOMEM
        assert sample(h, 0)[0] == 0
        assert var("live").value == whole, (i, var("live").value, whole)
        h.free()
    assert var("live").value == 0
    """)


def test_memory_for_the_factor_is_made_by_fp64_values(stub):
    """Blocks of 13 to 17 tiles keep a part of the factor in memory in FP64 values:
    FP32 values and gradients do not allocate it, a captured call and one that finds
    no memory do without it, and a gradient's buffers do not come with it."""
    _run(stub, """
    slots = 512 * 256 * 8  # workgroups, elements of a tile

    class Ptr:
        def __init__(self, a):
            self.a = a
        def data_ptr(self):
            return self.a.ctypes.data

    th, out = Ptr(theta), Ptr(np.zeros(1))
    for joint, ntm in ((200, 14), (250, 16), (272, 17)):
        tiles = slots * ntm * (ntm + 1) // 2
        h = handle(joint, 600)
        base = var("live").value
        sbv.sbv_loglik(h, theta, 5, sbv.SBV_FP32)
        assert var("live").value - base < 1 << 20
        calls = var("calls").value
        var("capturing").value = 1
        sbv.sbv_loglik_dev(h, th, 5, out, stream=1)
        var("capturing").value = 0
        assert var("calls").value == calls
        sbv.sbv_loglik_dev(h, th, 5, out, stream=1)
        assert tiles <= var("live").value - base < tiles + (1 << 20), (joint, var("live").value - base, tiles)
        calls = var("calls").value
        sbv.sbv_loglik(h, theta, 5)
        sbv.sbv_loglik(h, theta, 5, sbv.SBV_FP32)
        assert var("calls").value == calls
        h.free()

        h = handle(joint, 600)
        launches = var("launches").value
        var("max_bytes").value = 1 << 24
        sbv.sbv_loglik(h, theta, 5)
        refused = var("calls").value
        sbv.sbv_loglik(h, theta, 5)
        assert var("calls").value == refused and var("launches").value > launches
        var("max_bytes").value = -1
        h.free()
    assert var("live").value == 0
    """)
