"""Top-K select and significance counts at the edges of their kernels: how many radix passes the
select needs, the candidate limit, query tiles and the direct count's limit. Everything is exact:
indices, score bits and counts equal numpy's."""
from __future__ import annotations

import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stt():
    import paper_1401_8060_amd.stt as stt
    return stt


@pytest.fixture(scope="module")
def ctx(stt):
    c = stt.Context(0)
    yield c
    c.close()


def _say(*a):
    print(*a, flush=True, file=sys.stderr)


def _scores(kind, n):
    rng = np.random.default_rng(n)
    if kind == "normal":
        z = rng.standard_normal(n)
    elif kind == "equal":  # ties to the last index bit: every pass runs
        z = np.full(n, 1.5)
    elif kind == "nan":
        z = np.full(n, np.nan)
    elif kind == "two":    # more equal scores than candidates
        z = np.where(rng.random(n) < 0.5, 2.0, 1.0)
    else:                  # neighbouring floats: the last score digit decides
        z = np.float32(1.0) + rng.integers(0, 4096, n) * np.float32(2.0 ** -23)
    return z.astype(np.float32)


@pytest.mark.parametrize("n", [1, 255, 2049, 16383, 16384, 16385, 70_001])
@pytest.mark.parametrize("kind", ["normal", "equal", "nan", "two", "near"])
def test_topk_edges(stt, ctx, kind, n):
    import torch
    z = _scores(kind, n)
    key = np.where(np.isnan(z), -np.inf, z)
    order = np.lexsort((np.arange(n), -key))
    dev = torch.from_numpy(z).cuda()
    for K in sorted({1, min(n, 1000), min(n, 8192)}):
        _say("topk", kind, n, K)
        idx, val = ctx.topk(dev, K, first=7)
        want = order[:K]
        assert np.array_equal(idx.cpu().numpy() - 7, want)
        assert np.array_equal(val.cpu().numpy(), key[want].astype(np.float32))


def _keys(stt, z, j):
    return np.array([stt.key_encode(float(a), int(b)) for a, b in zip(z, j)], dtype=np.uint64)


@pytest.mark.parametrize("n_bg,n_fg", [(511, 3), (512, 300), (513, 1), (513, 64), (513, 65), (9000, 4095), (9000, 4096),
                                       (9000, 4097), (20_000, 9001), (100_003, 7)])
def test_significance_edges(stt, ctx, n_bg, n_fg):
    """Counts with many ties and empty keys on both sides, around the tile size and the direct limit."""
    import torch
    _say("significance", n_bg, n_fg)
    rng = np.random.default_rng(n_bg + n_fg)
    kb = _keys(stt, rng.standard_normal(n_bg).round(1), rng.integers(0, 1000, n_bg))
    kf = _keys(stt, rng.standard_normal(n_fg).round(1), rng.integers(0, 1000, n_fg))
    kb[rng.random(n_bg) < 0.01] = 0
    kf[rng.random(n_fg) < 0.01] = 0
    hb, hf = kb >> np.uint64(32), kf >> np.uint64(32)
    want = n_bg - np.searchsorted(np.sort(hb), hf, side="left")
    alpha = 0.05
    cnt, fap, za = ctx.significance(torch.from_numpy(kb.view(np.int64)).cuda(), torch.from_numpy(kf.view(np.int64)).cuda(),
                                    alpha=alpha)
    assert np.array_equal(cnt.cpu().numpy(), want)
    assert np.array_equal(fap.cpu().numpy(), (want / n_bg).astype(np.float32))
    m = max(1, int(np.ceil(alpha * n_bg)))
    z = np.array([stt.key_decode(int(k))[0] if k else -np.inf for k in kb], dtype=np.float32)
    assert za.item() == np.sort(z)[::-1][m - 1]
