"""The two forward branches of the smooth statistic's autograd binding: with and without a gradient
asked for, and what autograd refuses."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import synth
from tests.parity_util import to_dev

pytestmark = pytest.mark.gpu


def test_forward_branches_agree():
    import torch
    import paper_1401_8060_amd.stt as stt
    from paper_1401_8060_amd.autograd import smooth_snr
    print("autograd branches", flush=True, file=sys.stderr)
    T, F, n = 100, 60, 33
    c = stt.Context(0)
    m = stt.Map(*to_dev(*synth.noise_map(T, F, seed=9)))
    th, K = c.tracks_to_theta(c.make_tracks(stt.Gen(seed=2, min_len=2, dtau_max=10 ** 6), T, F, 0, n))
    w = torch.linspace(-2, 1, n, device="cuda")
    plain = smooth_snr(c, m, th, K)
    assert not plain.requires_grad
    leaf = th.clone().requires_grad_(True)
    with torch.no_grad():
        assert torch.equal(smooth_snr(c, m, leaf, K), plain)
    z = smooth_snr(c, m, leaf, K)
    assert torch.equal(z.detach(), plain)
    _, g = c.grad(m, th, K)
    for _ in range(2):  # a graph that is kept gives the same gradient again
        (got,) = torch.autograd.grad(z, leaf, w, retain_graph=True)
        assert torch.equal(got, w[:, None] * g)
    with torch.no_grad():
        leaf.add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(z, leaf, w)
    c.close()
