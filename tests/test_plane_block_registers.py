"""The assembly block that compares one bit plane (open_plane) writes its masks
before it has read all of its inputs in the cases where the two threshold bits
differ.  A caller may pass one value as the class mask and as the mask of
accepted (or open) sites: the block has to be given separate registers for them.
Checked on the code the compiler makes of such a caller."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_03676_amd", "csrc")

SOURCE = r"""
#include "pa_device.h"
__global__ void probe(const uint32_t* in, uint32_t* out, uint32_t tb)
{
    const uint32_t x[1] = {in[threadIdx.x]}, c[1] = {in[64 + threadIdx.x]}, other = in[128 + threadIdx.x];
    uint32_t acc[1] = {ACC}, open[1] = {OPEN};
    pa::dev::open_plane<1>(x, tb, c, acc, open);
    out[threadIdx.x] = acc[0];
    out[64 + threadIdx.x] = open[0];
}
"""


@pytest.mark.parametrize("acc,open_", [("c[0]", "other"), ("other", "c[0]"), ("c[0]", "c[0]")])
def test_class_mask_keeps_its_register(tmp_path, acc, open_):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, asm = str(tmp_path / "probe.hip"), str(tmp_path / "probe.s")
    with open(src, "w") as f:
        f.write(SOURCE.replace("ACC", acc).replace("OPEN", open_))
    subprocess.check_call([hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-S",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, src, "-o", asm], stderr=subprocess.DEVNULL)
    text = open(asm).read()
    block = text[text.index("s_cmp_lt_u32"):text.index("Lpa_plane_end", text.rindex("s_cmp_lt_u32"))]
    selects = re.findall(r"v_bitop3_b32 (v\d+), (v\d+), (v\d+), (v\d+) bitop3:0xca", block)
    merges = re.findall(r"v_bitop3_b32 (v\d+), (v\d+), (v\d+), (v\d+) bitop3:0xf4", block)
    assert len(selects) >= 2 and len(merges) >= 1
    written = {s[0] for s in selects} | {m[0] for m in merges}
    for dst, cls, _, _ in selects:
        assert cls not in written, (dst, cls)
