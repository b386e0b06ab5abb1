"""Register use of the sweep kernels, read from the metadata of the built
library.  A launch of one sweep of the register path (L <= 64) is bound by
memory, so a value that the compiler puts into scratch memory there costs as
much as the spins themselves: these kernels use none, and all fit eight waves
per SIMD (64 vector registers)."""
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1703_03676_amd", "libpa.so")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _code_objects(data):
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            yield at
        at = data.find(b"\x7fELF", at + 4)


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(LIB):
        pytest.skip("libpa.so is not built")
    data = open(LIB, "rb").read()
    out = {}
    for base in _code_objects(data):
        shoff, = struct.unpack_from("<Q", data, base + 40)
        size, count = struct.unpack_from("<HH", data, base + 58)
        for s in range(count):
            sh = base + shoff + s * size
            if struct.unpack_from("<I", data, sh + 4)[0] != SHT_NOTE:
                continue
            off, = struct.unpack_from("<Q", data, sh + 24)
            namesz, descsz, kind = struct.unpack_from("<III", data, base + off)
            if kind != NT_AMDGPU_METADATA:
                continue
            at = base + off + 12 + (namesz + 3) // 4 * 4
            for k in msgpack.unpackb(data[at:at + descsz], strict_map_key=False)["amdhsa.kernels"]:
                out[k[".name"]] = k
    return out


def test_register_path_sweeps_use_no_scratch_memory():
    seen = 0
    for name, k in _kernels().items():
        m = re.search(r"12sweep_kernelILi(16|32|64)ELb([01])ELi([012])E", name)
        if not m:
            continue
        seen += 1
        assert k[".private_segment_fixed_size"] == 0, (m.groups(), k[".private_segment_fixed_size"])
        assert k[".vgpr_count"] <= 64, (m.groups(), k[".vgpr_count"])
    assert seen >= 18  # three lattice sizes, two stores, three updates
