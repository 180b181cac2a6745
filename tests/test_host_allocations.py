"""CPU-only count of what the library asks of the device when a plan and a batch
are created: their host time is mostly device allocations and copies, so a plan
makes three allocations (constants, two twiddle tables) and one copy, and a
batch one of each for all of its tables, whatever its number of launches; and of
the bytes a plan holds, which at 2 and 4 limbs have no padding.

The HIP runtime's calls are counted by a small stand-in, preloaded into a child
process, that gives out host memory and launches nothing."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stdlib.h>
#include <string.h>
int stub_allocs, stub_copies, stub_frees, stub_bytes;
int hipMalloc(void** p, size_t n) { stub_allocs++; stub_bytes += n; *p = malloc(n); return *p == 0 ? 2 : 0; }
int hipFree(void* p) { if (p) stub_frees++; free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; stub_copies++; memcpy(d, s, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipLaunchKernel(const void* f, ...) { (void)f; return 0; }
int __hipPushCallConfiguration(long a, int b, long c, int d, size_t e, void* s) {
  (void)a; (void)b; (void)c; (void)d; (void)e; (void)s; return 0; }
int __hipPopCallConfiguration(void* g, void* b, size_t* n, void** s) {
  memset(g, 0, 12); memset(b, 0, 12); *n = 0; *s = 0; return 0; }
static void* made(void) { return malloc(1); }
int hipStreamCreate(void** s) { *s = made(); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = made(); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamBeginCapture(void* s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = made(); return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = made(); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipGraphInstantiate(void** x, void* g, void* n, void* l, size_t s) {
  (void)g; (void)n; (void)l; (void)s; *x = made(); return 0; }
int hipGraphDestroy(void* g) { free(g); return 0; }
int hipGraphExecDestroy(void* g) { free(g); return 0; }
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
import moma_inputs as mi
import paper_2501_07535_amd as moma
lib, stub = moma.library(), ctypes.CDLL(sys.argv[2])
counts = [ctypes.c_int.in_dll(stub, n) for n in ("stub_allocs", "stub_copies", "stub_frees", "stub_bytes")]
def counted(f):
    for c in counts: c.value = 0
    assert f() == 0
    return [c.value for c in counts]
def words(v, L): return (ctypes.c_uint32 * L)(*[(v >> (32 * j)) & 0xFFFFFFFF for j in range(L)])
fields = [mi.find_prime(lam, 0) for lam in (64, 128, 256, 384)]
roots = [f.root(1 << 12) for f in fields]
for f, w in zip(fields, roots):
    print("plan", *counted(lambda: lib.moma_ntt_prepare(words(f.q, f.limbs), words(w, f.limbs), 1 << 12, f.limbs)))
class Fake:  # a job's data is never touched: nothing is launched
    pass
u32p = ctypes.POINTER(ctypes.c_uint32)
keep, jobs = [], []
for kind in (moma.JOB_FORWARD, moma.JOB_INVERSE, moma.JOB_VMUL):
    for f, w in zip(fields, roots):
        q, om = words(f.q, f.limbs), words(w, f.limbs)
        keep += [q, om]
        jobs.append(moma._Job(ctypes.cast(q, u32p), ctypes.cast(om, u32p), 1 << 12, f.limbs, int(kind), 0x1000, 0x2000,
                              0x3000, None))
h = ctypes.c_void_p()
arr = (moma._Job * len(jobs))(*jobs)
print("batch", *counted(lambda: lib.moma_batch_create(arr, len(jobs), ctypes.byref(h))))
print("destroy", *counted(lambda: lib.moma_batch_destroy(h)))
lib.moma_shutdown.restype = None
print("shutdown", *counted(lambda: lib.moma_shutdown() or 0))
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc is not available")
def test_plans_and_batches_are_created_with_few_allocations(tmp_path):
    stub = str(tmp_path / "libstub.so")
    (tmp_path / "stub.c").write_text(STUB)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-w", "-o", stub, str(tmp_path / "stub.c")])
    (tmp_path / "child.py").write_text(CHILD)
    env = dict(os.environ, MOMA_NO_COSTMODEL="1")
    env["LD_PRELOAD"] = ":".join([stub] + ([env["LD_PRELOAD"]] if env.get("LD_PRELOAD") else []))
    r = subprocess.run([sys.executable, str(tmp_path / "child.py"), ROOT, stub], env=env, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    rows = [l.split() for l in r.stdout.splitlines() if l.split()[0] in ("plan", "batch", "destroy", "shutdown")]
    got = {}
    for name, *v in rows:
        got.setdefault(name, []).append([int(x) for x in v])
    assert len(got["plan"]) == 4 and all(v[:2] == [3, 1] for v in got["plan"]), got
    assert [v[:3] for v in got["batch"]] == [[1, 1, 0]], got
    assert got["destroy"] == [[0, 0, 1, 0]] and got["shutdown"] == [[0, 0, 12, 0]], got
    # two tables of 2^12 entries: twice the digits (3, 5, 9 and 14 of 29 bits), padded
    # to whole 16 bytes above 4 limbs only; the rest is the constants
    for L, digits, padded, v in zip((2, 4, 8, 12), (3, 5, 9, 14), (6, 10, 20, 28), got["plan"]):
        consts = 4 * (4 * digits + 2 * 14 * L)
        assert v[3] == 2 * 4 * padded * (1 << 12) + consts, (L, v)
