"""The adaptive step's bisection decides from quickly computed overlaps where
they are far enough from the target: its result has to be the one of the plain
bisection on the exact overlap, bit for bit, on any histogram."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_03676_amd", "csrc")

SOURCE = r"""
#include "pa_host.h"
using namespace pa::host;

extern "C" int fast(const uint32_t* n, int bmin, int bmax, int N, long R, long Rprev, double beta, double beta_f,
                    double star, double* out, double* alpha)
{
    const Hist h{n, bmin, bmax, N};
    std::vector<double> w;
    return adapt_beta(h, R, Rprev, beta, beta_f, star, out, alpha, w) ? 1 : 0;
}

extern "C" int plain(const uint32_t* n, int bmin, int bmax, int N, long R, long Rprev, double beta, double beta_f,
                     double star, double* out, double* alpha)
{
    const Hist h{n, bmin, bmax, N};
    std::vector<double> w;
    if (overlap(h, R, Rprev, beta_f - beta, w) >= star) {
        *out = beta_f;
        *alpha = overlap(h, R, Rprev, beta_f - beta, w);
        return 1;
    }
    double lo = beta, hi = beta_f;
    for (int it = 0; it < 50; ++it) {
        const double mid = lo + 0.5 * (hi - lo);
        if (overlap(h, R, Rprev, mid - beta, w) >= star) lo = mid; else hi = mid;
    }
    if (lo == beta) return 0;
    *out = lo;
    *alpha = overlap(h, R, Rprev, lo - beta, w);
    return 1;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h") or not shutil.which("g++"):
        pytest.skip("no HIP headers or compiler")
    d = tmp_path_factory.mktemp("adapt")
    src, lib = str(d / "adapt.cpp"), str(d / "adapt.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call(["g++", "-O3", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, src, "-o", lib])
    return ctypes.CDLL(lib)


def _call(f, hist, N, R, beta, beta_f, star):
    occupied = np.nonzero(hist)[0]
    out, alpha = ctypes.c_double(-1.0), ctypes.c_double(-1.0)
    rc = f(hist.ctypes.data_as(ctypes.c_void_p), int(occupied[0]), int(occupied[-1]), N, ctypes.c_long(R),
           ctypes.c_long(int(hist.sum())), ctypes.c_double(beta), ctypes.c_double(beta_f), ctypes.c_double(star),
           ctypes.byref(out), ctypes.byref(alpha))
    return rc, out.value, alpha.value


@pytest.mark.parametrize("L", [4, 16, 64, 128, 256])
def test_same_step_as_the_plain_bisection(host, L):
    rng = np.random.default_rng(L)
    N = L * L
    for trial in range(6 if L >= 128 else 40):
        R = int(rng.integers(1, 100000 if trial % 2 else 300))
        hist = np.zeros(N + 1, np.uint32)
        if trial % 5 == 0:  # two separated peaks
            bins = np.concatenate([rng.integers(0, N // 8 + 1, R // 2 + 1), rng.integers(N // 2, N + 1, R // 2 + 1)])
        elif trial % 5 == 1:  # one bin
            bins = np.full(R, rng.integers(0, N + 1))
        else:
            bins = np.clip(np.round(rng.normal(rng.uniform(0.1, 0.6) * N, rng.uniform(0.3, 1.0) * L, R)), 0, N)
        np.add.at(hist, bins.astype(np.int64), 1)
        target = max(1, int(hist.sum() + rng.integers(-20, 21)))
        beta = float(rng.uniform(0.0, 0.9))
        for beta_f in (beta + 1e-9, beta + float(rng.uniform(0.0, 0.01)), 1.0, 40.0, beta):
            for star in (0.5, 0.85, 0.999999, 1e-12, float(rng.uniform(0.01, 0.99))):
                assert _call(host.fast, hist, N, target, beta, beta_f, star) == \
                    _call(host.plain, hist, N, target, beta, beta_f, star)


def test_target_at_an_exact_overlap(host):
    # the target equals the overlap at a point of the bisection: the comparison
    # falls inside the margin and has to come out as equality
    rng = np.random.default_rng(7)
    N, R = 4096, 20000
    hist = np.zeros(N + 1, np.uint32)
    np.add.at(hist, np.clip(np.round(rng.normal(1200, 45, R)), 0, N).astype(np.int64), 1)
    for k in (6, 9, 14):
        beta_f = 0.3 + 2.0 ** -k
        for star in np.linspace(0.2, 0.95, 7):
            rc, out, alpha = _call(host.plain, hist, N, R, 0.3, 1.0, float(star))
            assert rc == 1
            assert _call(host.fast, hist, N, R, 0.3, 1.0, alpha) == _call(host.plain, hist, N, R, 0.3, 1.0, alpha)
            assert _call(host.fast, hist, N, R, 0.3, beta_f, alpha) == _call(host.plain, hist, N, R, 0.3, beta_f, alpha)
