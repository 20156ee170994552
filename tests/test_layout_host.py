"""The scorers' layout arithmetic (dev_common.hpp), compiled for the host and checked without a GPU."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("layout") / "layout"
    src = os.path.join(ROOT, "tests", "helpers", "layout_host.cpp")
    subprocess.run([hipcc, "-O2", "-x", "hip", "--offload-arch=gfx950", "-w",
                    "-I", os.path.join(ROOT, "paper_1401_8060_amd", "csrc"), src, "-o", str(out)],
                   check=True, capture_output=True)

    def run(lines):
        r = subprocess.run([str(out)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return r.stdout.strip().split("\n")
    return run


@pytest.mark.parametrize("nb", [1, 2, 3, 4, 5, 7, 8, 63, 64, 65, 125, 126, 127, 128])
def test_bucket_numbers_are_a_bijection(layout, nb):
    """Every (extent, start) has its own number in [0, nb (nb + 1) / 2), longest class first; within
    a class numbers go by start, then by extent."""
    cw = int(layout([f"class {nb}"])[0])
    assert cw >= 1 and -(-nb // cw) <= 4
    pairs = [(e, b0) for e in range(nb) for b0 in range(e + 1)]
    num = [int(x) for x in layout([f"bucket {e} {b0} {cw} {nb}" for e, b0 in pairs])]
    assert sorted(num) == list(range(len(pairs)))
    by_number = [p for _, p in sorted(zip(num, pairs))]
    assert by_number == sorted(pairs, key=lambda p: (p[0] // cw, p[1], p[0]))
