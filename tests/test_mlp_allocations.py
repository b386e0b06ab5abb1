"""The step proposer takes all of its host memory when it is created: a gradient
or a training call makes no pinned memory and no event of its own, so it is no
slower the first time and cannot fail for them.  The host part of pa_mlp.hip is
compiled alone and linked to a stand-in for the HIP runtime that counts (its
kernels do nothing)."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_03676_amd", "csrc")

RUNTIME = r"""
#include <stddef.h>
#include <stdlib.h>
#include <string.h>
char FATBIN[64];
int made = 0, freed = 0, uploads = 0, launches = 0;
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; ++made; *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void* p) { ++freed; free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned f) { (void)f; *d = h; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; ++made; *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { ++freed; free(e); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return ""; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st)
{ (void)st; if (k == 1) ++uploads; memcpy(d, s, n); return 0; }
struct dim { unsigned x, y, z; };
int hipLaunchKernel(const void* f, struct dim g, struct dim b, void** a, size_t m, void* s)
{ (void)f; (void)g; (void)b; (void)a; (void)m; (void)s; ++launches; return 0; }
int __hipPushCallConfiguration(struct dim g, struct dim b, size_t m, void* s)
{ (void)g; (void)b; (void)m; (void)s; return 0; }
int __hipPopCallConfiguration(struct dim* g, struct dim* b, size_t* m, void** s)
{ (void)g; (void)b; (void)m; (void)s; return 0; }
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipRegisterFunction(void** h, const void* f, char* d, const char* n, unsigned t, void* a, void* b, void* c,
                           void* e, int* w)
{ (void)h; (void)f; (void)d; (void)n; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not shutil.which("gcc"):
        pytest.skip("no compiler")
    d = tmp_path_factory.mktemp("mlp")
    obj, rt, so = str(d / "mlp.o"), str(d / "rt.c"), str(d / "mlp.so")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-c",
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "pa_mlp.hip"),
                           "-o", obj], stderr=subprocess.DEVNULL)
    undefined = subprocess.check_output(["nm", "-u", obj]).decode()
    names = re.findall(r"\b(__hip_fatbin\w*)", undefined) or ["unused_fatbin"]
    with open(rt, "w") as f:
        f.write(RUNTIME.replace("FATBIN", names[0]))
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", rt, obj, "-lstdc++", "-lm", "-o", so])
    h = ctypes.CDLL(so)
    h.pa_mlp_workspace_bytes.restype = ctypes.c_size_t
    return h


def _count(lib, name):
    return ctypes.c_int.in_dll(lib, name).value


@pytest.mark.parametrize("max_batch", [1, 64, 512, 20000])
def test_calls_make_no_host_memory(lib, max_batch):
    vp = ctypes.c_void_p
    nbytes = lib.pa_mlp_workspace_bytes(max_batch)
    raw = np.zeros(nbytes + 256, np.uint8)
    ws = raw.ctypes.data + (-raw.ctypes.data) % 256
    made0, freed0 = _count(lib, "made"), _count(lib, "freed")
    m = vp()
    assert lib.pa_mlp_create(max_batch, ctypes.c_uint64(3), vp(ws), ctypes.c_size_t(nbytes), vp(0),
                             ctypes.byref(m)) == 0
    made, freed = _count(lib, "made"), _count(lib, "freed")
    n = 50000
    x, t = np.zeros((n, 8), np.float32), np.zeros(n, np.float32)
    grad, loss = np.zeros(4801, np.float32), ctypes.c_float()
    for _ in range(2):
        assert lib.pa_mlp_gradient(m, vp(x.ctypes.data), vp(t.ctypes.data), max_batch, vp(grad.ctypes.data),
                                   ctypes.byref(loss)) == 0
    for samples, epochs in ((max_batch, 1), (n, 3), (max_batch, 2000 if max_batch <= 512 else 3)):
        losses = np.full(epochs, np.nan, np.float32)
        launches = _count(lib, "launches")
        assert lib.pa_mlp_train(m, vp(x.ctypes.data), vp(t.ctypes.data), samples, max_batch, epochs,
                                ctypes.c_float(0.01), ctypes.c_float(0.9), ctypes.c_uint64(1),
                                vp(losses.ctypes.data)) == 0
        assert np.all(losses == 0.0)  # every epoch's loss was written
        assert _count(lib, "launches") >= launches + 2 * epochs * (samples // max_batch)
    assert (_count(lib, "made"), _count(lib, "freed")) == (made, freed)
    assert lib.pa_mlp_free(m) == 0
    assert _count(lib, "made") - made0 == _count(lib, "freed") - freed0
