"""The smooth statistic's gathers of an FP32 map, read from the gfx950 assembly of the present code.

The two columns of a sample are loaded back to back, by array: the second column's lines are the first one's of the
neighbouring lane, and leave the L1 when other work comes in between."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_gathers_go_out_back_to_back(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path / "smooth.s"
    subprocess.run([hipcc, "--cuda-device-only", "-S", "-O3", "-std=c++17", "--offload-arch=gfx950", "-w",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1401_8060_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "smooth.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    body = re.search(r"^_ZN3stt13k_smooth_grad\w+:(.*?)^\s*s_endpgm", out.read_text(), re.S | re.M)[1]
    ops = [x.strip().split()[0] for x in body.split("\n") if re.match(r"\s+[a-z]\w*_\w+", x)]
    at = [i for i, op in enumerate(ops) if op.startswith("global_load")]
    assert [ops[i] for i in at] == ["global_load_dwordx2"] * 2 + ["global_load_dwordx4"] * 2
    assert at[1] - at[0] <= 2 and at[3] - at[2] <= 2 and at[3] - at[0] <= 8, at
