"""Sums exchanged between the lanes of a wave through LDS: the order of the stores and loads is stated.

The builtin for a wave barrier keeps instructions from moving across it but says nothing about memory. The
compiler has to be told, by a fence at wavefront scope on each side, that other lanes' stores come first."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_wave_barriers_lie_between_fences(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path / "md_wave.ll"
    subprocess.run([hipcc, "--cuda-device-only", "-S", "-emit-llvm", "-O3", "-std=c++17", "--offload-arch=gfx950", "-w",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1401_8060_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "md_wave.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    ir = [x.strip() for x in out.read_text().split("\n") if x.strip()]
    at = [i for i, x in enumerate(ir) if re.search(r"call void @llvm\.amdgcn\.wave\.barrier", x)]
    assert len(at) >= 2  # before the sums are read and before the next round writes
    for i in at:
        assert ir[i - 1].startswith('fence syncscope("wavefront') and "release" in ir[i - 1], ir[i - 2: i + 2]
        assert ir[i + 1].startswith('fence syncscope("wavefront') and "acquire" in ir[i + 1], ir[i - 2: i + 2]
