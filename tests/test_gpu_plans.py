"""Plans of the scorers that the other tests pass by: padded map rows, polynomial cosines, and free-t_mid and
delay-grid calls that read the caller's FP32 map unfolded.

Routes agree bit for bit; scores agree with the FP64 oracle to the scorers' tolerance (1e-5)."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import synth
from tests.parity_util import assert_close, key_to_host

pytestmark = pytest.mark.gpu

DT = 2684355


@pytest.fixture(scope="module")
def stt():
    import paper_1401_8060_amd.stt as stt
    return stt


def _say(*a):
    print(*a, flush=True, file=sys.stderr)


def _padded(stt, T, F, pad, seed):
    """A map of F rows in columns of F + pad, the padding full of values that no scorer may use."""
    import torch
    Y, s = synth.noise_map(T, F, seed=seed, sigma=("loguniform", 0.5, 2.0))
    Yp = np.full((T, F + pad), 1e30 + 1e30j, np.complex64)
    sp = np.full((T, F + pad), 1e-30, np.float32)
    Yp[:, :F], sp[:, :F] = Y, s
    return stt.Map(torch.from_numpy(Yp).cuda()[:, :F], torch.from_numpy(sp).cuda()[:, :F]), Y, s


def _i32(*t):
    return [x.cpu().numpy().view(np.int32) for x in t]


@pytest.mark.parametrize("hw", [True, False], ids=["hw", "poly"])
@pytest.mark.parametrize("T,F,pad,n", [(60, 41, 3, 5000), (520, 500, 1, 700), (300, 700, 5, 100_000)])
def test_padded_rows_and_polynomial_cosines(orc, stt, T, F, pad, n, hw):
    """Every route of a plain search, by path and by size, on padded columns and in FP16."""
    _say("plans", T, F, pad, n, hw)
    m, Y, s = _padded(stt, T, F, pad, 70 + T)
    g = stt.Gen(seed=5, min_len=10, dtau_max=DT)
    c = stt.Context(0)
    c.set_trig(hw)
    z_orc = orc.score_gen(orc.Map(Y, s), 5, 0, 10, DT, 0, min(n, 5000))
    for mm in (m, c.pack_p16(m)):
        got = []
        for path in (0, 1, 2, 3):
            c.set_path(path)
            z, key = c.score(mm, gen=g, n=n)
            zd, mi, _ = c.score_maxdelay(mm, -DT, DT // 4, 9, gen=g, n=n)
            got.append((_i32(z, zd, mi), key_to_host(key)))
        for a, key in got[1:]:
            assert all(np.array_equal(x, y) for x, y in zip(a, got[0][0])) and key == got[0][1]
        if mm is m:
            assert_close(got[0][0][0].view(np.float32)[:5000], z_orc, what=f"hw={hw}")
    c.set_path(0)
    keys = c.score_batch([m, m], g, [n, 300])  # map 0 draws the search's templates
    assert int(keys[0].item()) & 0xFFFFFFFFFFFFFFFF == key_to_host(c.score(m, gen=g, n=n)[1])
    c.close()


@pytest.mark.parametrize("T,F,n", [(500, 501, 300), (300, 900, 600), (1024, 300, 1171), (300, 900, 500)])
def test_small_calls_unfolded(orc, stt, T, F, n):
    """Lists of free-t_mid templates and of templates of the delay grid that gather from the caller's (padded) FP32
    map: (500, 501) and (1024, 300) by their columns, 600 of (300, 900) by their number; 500 of it fold first."""
    _say("unfolded", T, F, n)
    m, Y, s = _padded(stt, T, F, 7, 90 + T)
    c = stt.Context(0)
    g = stt.Gen(seed=8, min_len=10, dtau_max=DT)
    tm = c.make_tracks_tm(g, T, F, 0, n)
    z0 = _i32(c.score_tm(m, tracks=tm)[0])[0]
    c.set_path(2)
    z2, key2 = c.score_tm(m, gen=g, n=n)  # slabs, from the fold
    assert np.array_equal(z0, _i32(z2)[0])
    c.set_path(0)
    z, mi, _ = c.score_maxdelay(m, -DT, DT // 4, 8, gen=g, n=n)
    c.set_path(2)
    zs, ms, _ = c.score_maxdelay(m, -DT, DT // 4, 8, gen=g, n=n)
    assert all(np.array_equal(a, b) for a, b in zip(_i32(z, mi), _i32(zs, ms)))
    assert_close(z0.view(np.float32), orc.score_tm_gen_idx(orc.Map(Y, s), 8, 0, 10, DT, np.arange(n)),
                 what="free t_mid")
    c.close()
