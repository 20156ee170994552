"""Wait states around the slab scorers' LDS-DMA copies, read from the gfx950 assembly of the present code.

The copies are inline assembly, which the compiler's hazard pass does not look into: a wait state has to lie
between a scalar write of M0 (the LDS destination) and the copy, and a scalar register that a vector instruction
wrote may not be a copy's address within five wait states."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """Per kernel, its instructions in order: [(mnemonic, operands)]; labels as ("label", "")."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("dma") / "dma.s"
    subprocess.run([hipcc, "--cuda-device-only", "-S", "-O3", "-std=c++17", "--offload-arch=gfx950", "-w",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1401_8060_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "slab_dma.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    ins = []
    for line in out.read_text().split("\n"):
        line = line.split(";")[0].strip()
        if re.match(r"[.\w$]+:$", line):
            ins.append(("label", ""))
        elif re.match(r"[sv]_|global_|ds_|buffer_|scratch_", line):
            op, _, args = line.partition(" ")
            ins.append((op, args))
    return ins


def _copies(ins):
    return [i for i, (op, _) in enumerate(ins) if op.startswith("global_load_lds")]


def _sregs(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand.strip())
    return set(range(int(m[1]), int(m[2]) + 1)) if m else ({int(operand.strip()[1:])} if re.fullmatch(r"s\d+", operand.strip()) else set())


def test_wait_state_between_m0_and_copy(asm):
    at = _copies(asm)
    assert len(at) >= 8  # two staging kernels, and one copy loop per phase of the scorer
    for i in at:
        op, args = asm[i - 1]
        assert op != "label" and not args.startswith("m0"), asm[i - 3: i + 1]
        assert asm[i - 2][0] == "s_mov_b32" and asm[i - 2][1].startswith("m0"), asm[i - 3: i + 1]


def test_copy_address_is_scalar_written(asm):
    for i in _copies(asm):
        addr = _sregs(asm[i][1].split(",")[1])
        assert len(addr) == 2
        op, args = asm[i - 1]  # the address's last writer is a scalar instruction
        assert op.startswith("s_") and _sregs(args.split(",")[0]) == addr, asm[i - 3: i + 1]
