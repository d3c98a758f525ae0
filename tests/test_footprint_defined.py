"""An inactive pixel's footprint position is a defined value.

The kernels compare every lane's x0 and y0 wave-wide before they mask the
inactive lanes out, and a conversion of NaN, infinity or a float past the
integers' range is undefined: the compiler may drop whatever depends on it.
Compiled here for the GPU with such a coordinate as a constant, a kernel that
stores the position must still hold the store.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

SOURCE = """
#include "ctf_device.h"
extern "C" __global__ void k_foot(int* out, float4 d) { out[0] = ctf::footprint(%(u)s, %(v)s, d, 64.0f, 64.0f).%(axis)s; }
extern "C" __global__ void k_wave(int* out, float4 d) { out[0] = ctf::wave_footprint(%(u)s, %(v)s, d, 64.0f, 64.0f).%(axis)s; }
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("axis", ["x0", "y0"])
@pytest.mark.parametrize("bad", ['__builtin_nanf("")', "__builtin_inff()", "-1e30f"])
def test_position_of_an_inactive_pixel(tmp_path, axis, bad):
    src = tmp_path / "foot.hip"
    u, v = (bad, "0.25f") if axis == "x0" else ("0.25f", bad)
    src.write_text(SOURCE % {"u": u, "v": v, "axis": axis})
    ir = subprocess.run(
        [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off", "--offload-device-only", "-S",
         "-emit-llvm", "-I" + os.path.join(ROOT, "include"),
         "-I" + os.path.join(ROOT, "paper_2506_17770_amd", "csrc"), str(src), "-o", "-"],
        capture_output=True, text=True, check=True).stdout
    for kernel in ("k_foot", "k_wave"):
        body = ir[ir.index(f"@{kernel}("):]
        body = body[:body.index("\n}")]
        stores = [line for line in body.splitlines() if line.lstrip().startswith("store ")]
        assert stores and not any("poison" in s or "undef" in s for s in stores), body
