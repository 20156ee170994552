"""The scorers' layout arithmetic (dev_common.hpp), compiled for the host and checked without a GPU."""
from __future__ import annotations

import os
import shutil
import subprocess

import numpy as np
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


def _rows(Dt, f0, f1, f2):
    k = np.arange(Dt + 1, dtype=object)
    return [int(x) for x in ((Dt - k) ** 2 * f0 + 2 * (Dt - k) * k * f1 + k * k * f2) // (256 * Dt * Dt)]


def test_lazy_period_keeps_its_bound(layout):
    """R columns between seeds: R/2 2^-32 + 3 2^-38 < 2^-9 / Dt^2, and no smaller power of two than needed."""
    ds = [1, 9, 511, 512, 1020, 1021, 1022, 1439, 1440, 2023, 2024, 2025, 2829, 2830, 2831, 2895]
    got = [int(x) for x in layout([f"period {d}" for d in ds])]
    for d, r in zip(ds, got):
        ok = [R for R in (16, 8, 4, 2) if d * d * (32 * R + 3) < 2 ** 29]
        assert r == (ok[0] if ok else 1), d


@pytest.mark.parametrize("F", [1, 2, 151, 1000, 5000, 32767])
def test_lazy_and_exact_rows(layout, F):
    """Rows of both walks equal the integer floor of Eq. 6 at the longest extents of every seed period, with control
    points at the ends of the band and where numerators fall on multiples of the row size."""
    rng = np.random.default_rng(F)
    cases = []
    for Dt in (1, 2, 3, 9, 100, 511, 512, 999, 1020, 1021, 1022, 1439, 1440, 2023, 2024, 2830, 2831, 2895):
        lim = F * 256
        ctl = [(0, 0, lim - 1), (lim - 1, 0, lim - 1), (0, lim - 1, 0), (lim - 1, lim - 1, 0)]
        ctl += [tuple(int(x) for x in rng.integers(0, lim, 3)) for _ in range(6)]
        ctl += [tuple(int(x) // 256 * 256 for x in rng.integers(0, lim, 3)) for _ in range(4)]
        cases += [(Dt, *c) for c in ctl]
    R = [int(x) for x in layout([f"period {c[0]}" for c in cases])]
    lazy = layout([f"lazy {c[0]} {c[1]} {c[2]} {c[3]} {max(r, 1)}" for c, r in zip(cases, R)])
    exact = layout([f"exact {c[0]} {c[1]} {c[2]} {c[3]} {-(i % 40)}" for i, c in enumerate(cases)])
    for c, a, b in zip(cases, lazy, exact):
        want = _rows(*c)
        assert [int(x) for x in a.split()] == want, c
        assert [int(x) for x in b.split()] == want, c
