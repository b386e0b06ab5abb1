"""The key by which a batch finds a launch shape that was timed before tells
launches apart that hold different lattice sizes, however many waves they
have together, and not the order in which the runs are given."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_03676_amd", "csrc")

SOURCE = r"""
#include "pa_host.h"
static pa::host::LaunchMix mix(const int* L, const long* waves, int n)
{
    pa::host::LaunchMix m;
    for (int i = 0; i < n; ++i) m.add(L[i], waves[i]);
    return m.rounded();
}
extern "C" int same(const int* La, const long* wa, int na, const int* Lb, const long* wb, int nb)
{
    const pa::host::LaunchMix a = mix(La, wa, na), b = mix(Lb, wb, nb);
    return !(a < b) && !(b < a);
}
"""


@pytest.fixture(scope="module")
def same(tmp_path_factory):
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h") or not shutil.which("g++"):
        pytest.skip("no HIP headers or compiler")
    d = tmp_path_factory.mktemp("mix")
    src, lib = str(d / "mix.cpp"), str(d / "mix.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC, src, "-o", lib])
    f = ctypes.CDLL(lib).same

    def call(a, b):
        arrays = []
        for runs in (a, b):
            arrays += [(ctypes.c_int * len(runs))(*[L for L, _ in runs]),
                       (ctypes.c_long * len(runs))(*[w for _, w in runs]), len(runs)]
        return bool(f(*arrays))
    return call


def test_lattice_sizes_are_told_apart(same):
    sizes = (16, 32, 64, 128, 256)
    for L in sizes:
        for M in sizes:
            assert same([(L, 1000)], [(M, 1000)]) == (L == M)
    assert not same([(16, 500), (64, 500)], [(16, 1000)])
    assert not same([(16, 500), (64, 500)], [(64, 500), (32, 500)])


def test_runs_of_one_size_add_up_to_a_power_of_two(same):
    assert same([(16, 300), (64, 40), (16, 200)], [(64, 33), (16, 512)])
    assert not same([(16, 513)], [(16, 512)])
    assert same([(256, 1)], [(256, 1)]) and not same([(256, 1)], [(256, 2)])
