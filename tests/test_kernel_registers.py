"""Registers of kernels whose waves per SIMD depend on a few of them, from the
metadata of the built library (512 vector registers a lane of a SIMD, given out
in eights)."""
import os
import re
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_17770_amd", "libctf.so")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
NOTE = struct.pack("<I", 7)     # name "AMDGPU", then type 32: the kernels' metadata


@pytest.fixture(scope="module")
def kernels():
    """Mangled name -> metadata of every kernel of libctf.so."""
    if not os.path.exists(LIB):
        pytest.skip("libctf.so is not built")
    with open(LIB, "rb") as f:
        lib = f.read()
    found, at = {}, lib.find(BUNDLE)
    while at >= 0:
        n, p = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
        for _ in range(n):
            offset, size, idlen = struct.unpack_from("<QQQ", lib, p)
            p += 24 + idlen
            code = lib[at + offset:at + offset + size]
            name = code.find(b"AMDGPU\0")
            while name >= 0:
                if name >= 12 and code[name - 12:name - 8] == NOTE and struct.unpack_from("<I", code, name - 4)[0] == 32:
                    desc = struct.unpack_from("<I", code, name - 8)[0]
                    meta = msgpack.unpackb(code[name + 8:name + 8 + desc])
                    found.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
                name = code.find(b"AMDGPU\0", name + 7)
        at = lib.find(BUNDLE, at + 24)
    assert found
    return found


def test_full_filter_waves(kernels):
    """The bilinear full filter of a procedural texture: six waves per SIMD tap
    by tap, as many as 80 registers allow (3840x2160, 4096 wide: 306 us; 318 with
    five)."""
    seen = [k for n, k in kernels.items() if re.search(r"k_filter_simtILi0ELi0ELb0ELi0E", n)]
    assert seen
    for k in seen:
        assert k[".vgpr_count"] <= 80 and k[".vgpr_spill_count"] == 0, (k[".name"], k[".vgpr_count"])
