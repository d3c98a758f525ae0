"""The kernels' texel sets on the CPU: the device code of csrc/ctf_device.h,
compiled for the host with a wave's lanes as coroutines, against std::set.

Sorted row segments (boxes past the 16x16 window, one or two sets): counts,
the list in row-major order, each item written once, and each lane's first
items, over footprints that coincide, overlap by 1..F texels, touch, or lie at
the ends of the position range.  Windows (whole wave and half-waves): the set,
its count and every rank, from one texel to all 256.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_sets_of_a_wave(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "sets")
    emulation = os.path.join(HERE, "wave_emulation")
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-I" + emulation, "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2506_17770_amd", "csrc"), os.path.join(emulation, "sets.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
