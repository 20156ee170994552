"""The library's host side (stt_api.hip) with the HIP runtime replaced by a recorder: what it allocates and
launches, without a GPU."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RANKS = ["k_rank_sort:1", "k_rank_count:1", "k_rank_finish:1"]
DIRECT = ["k_count_louder:1"]


@pytest.fixture(scope="module")
def api(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("api") / "api"
    subprocess.run([hipcc, "--cuda-host-only", "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-w",
                    "-Xarch_host", "-fsanitize=signed-integer-overflow", "-Xarch_host",
                    "-fsanitize-trap=signed-integer-overflow", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1401_8060_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "api_host.cpp"), "-o", str(out)],
                   check=True, capture_output=True)

    def run(line):
        r = subprocess.run([str(out)], input=line + "\n", capture_output=True, text=True, check=True)
        return r.stdout.split()
    return run


@pytest.mark.parametrize("n_q,direct,ranks", [(1, 717, 718), (65, 759, 760), (1000, 1339, 1340), (4096, 3326, 3327),
                                              (100_000, 3326, 3327), (262_145, 3257, 3258), (1_000_000, 3900, 3901)])
def test_counts_take_ranks_where_they_are_faster(api, n_q, direct, ranks):
    """Both sides of the rule: references, for a number of queries, at which the sort of the queries pays."""
    assert all(x.startswith("k_count_louder:") for x in api(f"louder {direct} {n_q} 0 0 0 0")[2:])
    got = api(f"louder {ranks} {n_q} 0 0 0 0")
    assert got[:2] == ["0", "1"]
    assert [x.split(":")[0] for x in got[2:]] == [x.split(":")[0] for x in RANKS] * -(-n_q // 262_144)
    assert api(f"louder {ranks} {n_q} 9999999 0 0 0")[1] == "0"


@pytest.mark.parametrize("cap", [1, 2])
@pytest.mark.parametrize("have", [0, 9_999_999])
def test_captured_counts_use_no_scratch(api, cap, have):
    """A graph keeps the addresses it was captured with, and the scratch moves when a later call needs more of
    it: captured counts have to do without, also where it is large enough already (cap 2: the stream cannot be
    asked, as the null stream while another one captures)."""
    assert api(f"louder 1000 10 {have} {cap} 0 0") == ["0", "0", *DIRECT]


HIP_OOM, HIP_FAULT = 2, 719  # hipErrorOutOfMemory, hipErrorLaunchFailure
EHIP = "-4"  # STT_EHIP


def test_counts_without_memory_are_direct(api):
    """Out of memory leaves the direct counts, and no message of a failure that the caller never sees."""
    assert api(f"louder 1000 10 0 0 {HIP_OOM} 0") == ["0", "1", *DIRECT]


def test_counts_report_a_failed_stream(api):
    """The scratch waits for the stream before it moves; what the wait reports is the call's status."""
    assert api(f"louder 1000 10 64 0 0 {HIP_FAULT}") == [EHIP, "0", "message"]


def _slides(api, pairs, T=1000, F=1000):
    got = [int(x) for x in api(f"slides {T} {F} {len(pairs)} " + " ".join(f"{y} {s}" for y, s in pairs))]
    assert got[0] == 0 and sum(got[1:]) == len(pairs)
    return got[1:]


def test_slides_of_one_launch_write_distinct_buffers(api):
    """A launch writes its slides in no order, so slides into one buffer, of Y or of sigma, take launches of their
    own: the last one stands, as the calls order them."""
    own = [(k, k) for k in range(150)]
    assert _slides(api, own) == [64, 64, 22]
    assert _slides(api, [(0, 0), (0, 0), (1, 1), (2, 0), (2, 2), (3, 3)]) == [1, 2, 1, 2]
    assert _slides(api, [(k, 7) for k in range(5)]) == [1] * 5        # one sigma for all
    assert _slides(api, own[:64] + own[:64]) == [64, 64]              # the buffers of the launch before
    assert _slides(api, own[:63] + own[:1] + own[63:80]) == [63, 18]


@pytest.mark.parametrize("bytes_before", [8, 1400, 50_000, 300_000])
def test_captured_topk_after_any_other_call(api, bytes_before):
    """The select and the other users of the auxiliary scratch (packing, follow-up ranks) share it: whichever comes
    first, a select recorded later allocates nothing."""
    assert api(f"topk {bytes_before} 5000 10 1") == ["0", "0"]
    assert api("topk 0 5000 10 0") == ["0", "1"]


K160, K80 = 160 * 1024, 80 * 1024


def test_default_budget_leaves_the_shape_to_the_calls(api):
    """lds_bytes = 163840 is the documented default: setting it, alone or after another budget, is the context as it
    was created. A shape that was set stays."""
    def shape(sets, wg=0, tpt=0):
        return [int(x) for x in api(f"shape {wg} {tpt} {' '.join(map(str, sets))} - 10000000 8192")]
    free = shape([])
    assert free == [1024, 2, K80]
    assert shape([0]) == free and shape([K160]) == free
    assert shape([48 * 1024]) == [1024, 4, 48 * 1024]
    assert shape([48 * 1024, 0]) == [1024, 4, 48 * 1024]
    assert shape([48 * 1024, K160]) == free
    assert shape([K160], 1024, 4) == [1024, 4, K160] and shape([K80, K160], 512, 2) == [512, 2, K160]


@pytest.mark.parametrize("n0,n1", [(2**63 - 1, 2**63 - 1), (2**62, 2**62), (100, 2**32 + 1), (-1, 2**63 - 1)])
def test_batch_counts_are_refused_without_overflow(api, n0, n1):
    """Counts out of range are summed for the shape before they are refused (this build traps where a signed sum
    overflows)."""
    assert api(f"batch {n0} {n1}") == ["-2"]


@pytest.mark.parametrize("per,n,run", [(1, 1, 256), (245, 3, 256), (256, 2, 256), (257, 2, 256), (700, 5, 256), (513, 1, 512),
                                       (1025, 64, 512)])
def test_slide_workgroups_in_runs(api, per, n, run):
    """Each workgroup of each slide once: run by run of the XCD's part, slide by slide within a run, front to back."""
    got = [int(x) for x in api(f"items {per} {n} {run}")]
    want = [(k, at) for r in range(0, per, run) for k in range(n) for at in range(r, min(r + run, per))]
    assert list(zip(got[::2], got[1::2])) == want


@pytest.mark.parametrize("T,F,e,n,L,n_tau,want", [
    # measured times in us at the right: lane, slabs, wave
    (100, 128, 8, 5_000, 10, 8, "wave"),         # 34, 76, 25
    (100, 128, 8, 100_000, 10, 8, "lane"),       # 38, 77, 235
    (300, 300, 8, 100_000, 150, 8, "lane"),      # 94, 151, 245
    (1000, 1000, 8, 100_000, 10, 8, "wave"),     # 360, 430, 274
    (1000, 1000, 8, 150_000, 500, 8, "slab"),    # 629, 427, 572
    (1000, 1000, 8, 200_000, 10, 8, "slab"),     # 651, 421, 530
    (1000, 1000, 8, 150_000, 500, 17, "slab"),   # slabs 1237, wave 1692
    (500, 151, 8, 150_000, 10, 24, "slab"),      # 629, 532, 1084
    (700, 200, 8, 130_000, 10, 32, "lane"),      # lane 805, slabs 960
    (700, 1400, 8, 80_000, 10, 12, "wave"),      # wave 416, slabs 659
    (1900, 1900, 8, 130_000, 237, 32, "slab"),   # wave 5558, slabs 3630
    (1900, 1900, 4, 130_000, 237, 32, "slab"),   # wave 4091, slabs 3410
])
def test_delay_grid_scorer_by_cost(api, T, F, e, n, L, n_tau, want):
    assert api(f"md {T} {F} {e} {n} {L} {n_tau}") == [want]


@pytest.mark.parametrize("T,F,e,n,L,want", [
    # measured times in us at the right: slabs, wave
    (1000, 1000, 8, 100_000, 10, "wave"),        # 345, 306
    (1000, 1000, 8, 150_000, 10, "slab"),
    (1400, 1400, 8, 100_000, 175, "slab"),       # 584, 687
    (1400, 1400, 4, 100_000, 700, "slab"),       # 476, 597
    (1900, 1900, 8, 125_000, 237, "slab"),       # 970, 1411
    (1900, 1900, 4, 60_000, 1898, "slab"),       # 735, 949
    (2800, 2000, 8, 125_000, 2798, "slab"),      # 1453, 5138
    (1900, 1900, 8, 30_000, 10, "wave"),
    (20, 20, 8, 4095, 18, "wave"),
])
def test_free_tmid_scorer_by_cost(api, T, F, e, n, L, want):
    assert api(f"tm {T} {F} {e} {n} {L}") == [want]


@pytest.mark.parametrize("T,F,p16,wave,n,launches,want", [
    (300, 1000, 0, 1, 511, 1, 0), (300, 1000, 0, 1, 512, 1, 1), (499, 1000, 0, 1, 100, 1, 0), (500, 1000, 0, 1, 100, 1, 1),
    (1000, 1000, 0, 1, 1000, 1, 1), (1000, 1000, 0, 1, 1000, 2, 0), (1000, 1000, 0, 1, 1201, 1, 0),
    (500, 499, 0, 1, 1000, 1, 0), (1025, 1000, 0, 1, 100, 1, 0), (1000, 1000, 0, 0, 1000, 1, 0), (300, 1000, 1, 0, 10, 3, 1),
    (200, 4000, 0, 1, 100, 1, 0), (400, 3000, 0, 1, 100, 1, 1), (400, 30000, 0, 1, 16, 1, 1), (1000, 3999, 0, 1, 100, 2, 0),
    (1000, 4000, 0, 1, 100, 2, 1),
])
def test_direct_calls_that_read_the_map_unfolded(api, T, F, p16, wave, n, launches, want):
    assert api(f"gather {T} {F} {p16} {wave} {n} {launches}") == [str(want)]


def test_sort_by_extent_alone_for_one_round_of_register_staging(api):
    """A workgroup per CU at most, staged through registers: one extent per class; else the four classes."""
    assert api("class 0 256 256 126") == ["1"] and api("class 0 257 256 126") == ["32"]
    assert api("class 1 1 256 126") == ["32"] and api("class 0 1 256 1") == ["1"]


def test_lanes_gather_one_pixel_at_a_time_on_large_maps(api):
    assert api("one 8192000 1000 70000 340") == ["0"] and api("one 8192000 1000 70000 667") == ["1"]
    assert api("one 8192000 1000 300000 340") == ["1"] and api("one 4194304 1000 300000 340") == ["0"]


@pytest.mark.parametrize("T", [2, 20, 100, 500, 1000, 2896])
def test_bench_names_the_scorer_that_runs(api, T):
    import bench
    ns = [1, 4095, 4096, -(-60_000_000 // T) - 1, -(-60_000_000 // T), 80_000 * T // (T + 600), 80_000 * T // (T + 600) + 1]
    assert [api(f"plain {T} {n}")[0] for n in ns] == [bench.plain_scorer(T, n) for n in ns]
