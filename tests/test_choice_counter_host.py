"""What the counter of the chosen temperatures counts (pa_batch_choice_stats):
the overlaps that the adaptive step compares with its target, one for beta_f and
50 for the halvings, however many of them it evaluates."""
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
extern "C" long counted(const uint32_t* n, int bmin, int bmax, int N, long R, double beta_f, double star, int alpha)
{
    const pa::host::Hist h{n, bmin, bmax, N};
    std::vector<double> w;
    double out = 0.0, a = 0.0;
    int64_t evals = 7;
    pa::host::adapt_beta(h, R, R, 0.25, beta_f, star, &out, alpha ? &a : nullptr, w, &evals);
    return (long)evals - 7;
}
"""


@pytest.fixture(scope="module")
def counted(tmp_path_factory):
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h") or not shutil.which("g++"):
        pytest.skip("no HIP headers or compiler")
    d = tmp_path_factory.mktemp("count")
    src, lib = str(d / "count.cpp"), str(d / "count.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, src, "-o", lib])
    f = ctypes.CDLL(lib).counted
    f.restype = ctypes.c_long
    return f


@pytest.mark.parametrize("beta_f,star,alpha,expected", [(0.2501, 0.85, 0, 1), (1.0, 0.85, 0, 51), (1.0, 0.85, 1, 52),
                                                        (1.0, 0.5, 0, 51)])
def test_comparisons(counted, beta_f, star, alpha, expected):
    rng = np.random.default_rng(3)
    N, R = 4096, 20000
    hist = np.zeros(N + 1, np.uint32)
    np.add.at(hist, np.clip(np.round(rng.normal(1200, 45, R)), 0, N).astype(np.int64), 1)
    occupied = np.nonzero(hist)[0]
    assert counted(hist.ctypes.data_as(ctypes.c_void_p), int(occupied[0]), int(occupied[-1]), N, ctypes.c_long(R),
                   ctypes.c_double(beta_f), ctypes.c_double(star), alpha) == expected
