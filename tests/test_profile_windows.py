"""Profiling windows against a HIP runtime made of the C library (the library's
host code runs on the CPU, device memory is host memory, launches do nothing).
A window that runs out of events: ttn_tdvp_step has to return its error, wherever
in a sequence of held-back contractions the event was wanted (an exception out
of a destructor would end the process).  A window whose events read otherwise
at every call: its launch records and its sums have to come from one reading."""
import os
import pathlib
import subprocess
import sys

import pytest

STUB = r"""
#include <stdlib.h>
#include <string.h>
static int g_events = -1;   /* events left; < 0: no limit */
void stub_events(int n) { g_events = n; }
int hipEventCreate(void **e) {
    if (g_events == 0) return 2;
    if (g_events > 0) --g_events;
    *e = malloc(1);
    return 0;
}
int hipEventDestroy(void *e) { free(e); return 0; }
static int g_reads;
int hipEventElapsedTime(float *t, void *a, void *b) { *t = 1.0f + 0.0078125f * (g_reads++ % 64); return 0; }
int hipEventRecord(void *e, void *s) { return 0; }
int hipFree(void *p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
const char *hipGetErrorString(int e) { return e ? "out of events" : "ok"; }
int hipGetLastError(void) { return 0; }
int hipLaunchKernel(const void *f, unsigned long long a, unsigned b, unsigned long long c, unsigned d, void **args,
                    size_t lds, void *s) { return 0; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { memset(d, v, n); return 0; }
int hipStreamSynchronize(void *s) { return 0; }
int __hipPushCallConfiguration(unsigned long long a, unsigned b, unsigned long long c, unsigned d, size_t e, void *s) { return 0; }
int __hipPopCallConfiguration(void *a, void *b, void *c, void *d) {
    memset(a, 0, 12); memset(b, 0, 12); memset(c, 0, sizeof(size_t)); memset(d, 0, sizeof(void *)); return 0; }
static void *bin;
void **__hipRegisterFatBinary(const void *d) { return &bin; }
void __hipRegisterFunction(void **m, const void *h, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w) {}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {}
void __hipUnregisterFatBinary(void **m) {}
"""

DRIVER = r"""
import ctypes as C, sys, types
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.modules["torch"] = types.ModuleType("torch")     # the HIP runtime is the stub's
import numpy as np
from paper_2210_03763_amd import ttn as T
from paper_2210_03763_amd import workload as W
L = T.lib()
w = W.make_random_drive(4, 4, 3, 16, 2, 0.01, 2, 3, plus_sites=tuple(range(16)), eps=0.0, precision=int(sys.argv[2]))
keep = []
cfg = T.make_config(w, keep)
n = C.c_size_t(0)
assert L.ttn_workspace_query(C.byref(cfg), C.byref(n)) == 0
buf = (C.c_char * (n.value + 4096))()
e = np.ascontiguousarray(w.seg_edges, dtype=np.float64)
om, de = (np.ascontiguousarray(a, dtype=np.float64) for a in (w.omega, w.delta))
z = np.zeros(2, np.int32)
"""

OUT_OF_EVENTS = r"""
failed = 0
for events in list(range(0, 64, 2)) + [100000]:          # the pool grows by pairs, in a handle of its own
    stub.stub_events(-1)
    h = C.c_void_p()
    assert L.ttn_init(C.byref(cfg), (C.addressof(buf) + 4095) // 4096 * 4096, n, None, C.byref(h)) == 0
    assert L.ttn_set_pulses(h, om.shape[1], T._dptr(e), T._dptr(om), T._dptr(de), 0, T._iptr(z), T._iptr(z), T._dptr(np.zeros(2))) == 0
    assert L.ttn_profile_begin(h) == 0
    stub.stub_events(events)
    rc = L.ttn_tdvp_step(h, 0.01, 1, None)
    if rc != 0 and "out of events" in L.ttn_last_error(h).decode():
        failed += 1
    stub.stub_events(-1)
    L.ttn_destroy(h)
print("out of events", failed, flush=True)
assert failed == 32
"""

ONE_READING = r"""
h = C.c_void_p()
assert L.ttn_init(C.byref(cfg), (C.addressof(buf) + 4095) // 4096 * 4096, n, None, C.byref(h)) == 0
assert L.ttn_set_pulses(h, om.shape[1], T._dptr(e), T._dptr(om), T._dptr(de), 0, T._iptr(z), T._iptr(z), T._dptr(np.zeros(2))) == 0
assert L.ttn_profile_begin(h) == 0 and L.ttn_tdvp_step(h, 0.01, 1, None) == 0
p = T.Profile()
assert L.ttn_profile_end(h, C.byref(p)) == 0
recs = (T.LaunchRec * L.ttn_profile_launches(h, None, 0))()
L.ttn_profile_launches(h, recs, len(recs))
single = sum(r.ms for r in recs if r.ms >= 0)
print("launches", len(recs), single + p.heff.ms, p.gemm_f32.ms + p.gemm_f64.ms, flush=True)
assert len(recs) == p.gemm_f32.launches + p.gemm_f64.launches
assert all((r.ms < 0) == (r.heff == 1) for r in recs)
assert abs(single + p.heff.ms - (p.gemm_f32.ms + p.gemm_f64.ms)) < 1e-9 * len(recs)
"""


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("body", [OUT_OF_EVENTS, ONE_READING], ids=["out-of-events", "one-reading"])
def test_window(tmp_path, body, precision):
    src, so, drv = tmp_path / "hip_stub.c", tmp_path / "libhip_stub.so", tmp_path / "driver.py"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(so), str(src)], check=True)
    drv.write_text(DRIVER + body)
    root = str(pathlib.Path(__file__).parents[1])
    r = subprocess.run([sys.executable, str(drv), str(so), str(precision)], capture_output=True, text=True, timeout=120,
                       cwd=root, env=dict(os.environ, PYTHONPATH=root))
    print(r.stdout[-500:], r.stderr[-1500:], flush=True)
    assert r.returncode == 0, f"exit {r.returncode}"
