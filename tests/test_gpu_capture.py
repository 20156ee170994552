"""Calls recorded in a HIP graph: replays give the eager call's results, also after later calls made the
context's scratch grow."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import synth
from tests.parity_util import to_dev

pytestmark = pytest.mark.gpu


def _keys(rng, n):
    z = np.abs(rng.standard_normal(n)).astype(np.float32)
    hi = z.view(np.uint32).astype(np.uint64) | np.uint64(0x80000000)
    return ((hi << np.uint64(32)) | (np.uint64(0xFFFFFFFF) - np.arange(n, dtype=np.uint64))).view(np.int64)


def test_captured_counts_survive_scratch_growth():
    import torch
    import paper_1401_8060_amd.stt as stt
    s = torch.cuda.Stream()
    c = stt.Context(0, s)
    rng = np.random.default_rng(2)
    with torch.cuda.stream(s):
        bg, fg = torch.from_numpy(_keys(rng, 3000)).cuda(), torch.from_numpy(_keys(rng, 700)).cuda()
        want = c.significance(bg, fg, alpha=None)[:2]
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            cnt, fap, _ = c.significance(bg, fg, alpha=None)
        m = stt.Map(*to_dev(*synth.noise_map(40, 32, seed=1)))
        for rep in range(3):
            print("captured counts, replay", rep, flush=True, file=sys.stderr)
            cnt.zero_()
            graph.replay()
            s.synchronize()
            assert torch.equal(cnt, want[0]) and torch.equal(fap, want[1])
            # a larger call between the replays
            c.score_maxdelay(m, 0, 1000, 2, gen=stt.Gen(seed=1, min_len=10, dtau_max=5), n=300_000 * (rep + 1), snr=None,
                            tau_idx=None)
            s.synchronize()
    c.close()


def test_topk_captured_after_packing():
    """Packing is the first user of the scratch that a recorded select shares."""
    import torch
    import paper_1401_8060_amd.stt as stt
    s = torch.cuda.Stream()
    c = stt.Context(0, s)
    with torch.cuda.stream(s):
        c.pack_p16(stt.Map(*to_dev(*synth.noise_map(40, 32, seed=1))))
        z = torch.randn(100_000, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            idx, val = c.topk(z, 100)
        for rep in range(3):
            print("captured select, replay", rep, flush=True, file=sys.stderr)
            z.normal_()
            graph.replay()
            s.synchronize()
            want = c.topk(z, 100)
            assert torch.equal(idx, want[0]) and torch.equal(val, want[1])
            assert val.tolist() == sorted(z.tolist(), reverse=True)[:100]
    c.close()
