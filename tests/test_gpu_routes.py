"""Every scorer gives the same bits, at the edges of what chooses between them: flush groups of 16
pixels, calls smaller than the map, wave-per-template launches that stride over more templates than
they have waves, the pixel thresholds between the scorers, and the slab shapes chosen by size."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import synth
from tests.parity_util import key_to_host, to_dev

pytestmark = pytest.mark.gpu

DT = 1234567


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


def _map(stt, T, F, seed=5):
    return stt.Map(*to_dev(*synth.noise_map(T, F, seed=seed, sigma=("loguniform", 0.5, 2.0))))


def _host(*t):
    return [x.view(dtype=x.dtype).cpu().numpy().view(np.int32) for x in t]


def _tracks(ctx, stt, T, F, n):
    """Tracks whose pixel counts run through every residue of 16, with invalid ones among them."""
    import torch
    tr = ctx.make_tracks(stt.Gen(seed=3, min_len=2, dtau_max=DT), T, F, 0, n).cpu().numpy()
    Ts = np.arange(n) % (T - 1) + 2
    tr[:, 0] = np.minimum(tr[:, 0], T - Ts)
    tr[:, 1] = tr[:, 0] + Ts - 1
    if n > 8:
        tr[7, 1] = T        # past the map: scores NaN
        tr[n - 1, 0] = -1
    return torch.from_numpy(tr).cuda()


@pytest.mark.parametrize("p16", [False, True], ids=["f32", "p16"])
@pytest.mark.parametrize("T,F", [(2, 3), (16, 40), (17, 40), (33, 64), (100, 128)])
def test_direct_scorers_at_group_edges(stt, ctx, T, F, p16):
    m = _map(stt, T, F)
    if p16:
        m = ctx.pack_p16(m)
    for n in (1, 3, 4, 5, F, F + 1, 4096, 4103):  # 4 templates a workgroup, 1024 workgroups: 4097 strides
        _say("routes", T, F, p16, n)
        tr = _tracks(ctx, stt, T, F, n)
        got = []
        for path in (3, 1, 0, 2):
            ctx.set_path(path)
            z, key = ctx.score(m, tracks=tr)
            got.append((*_host(z), key_to_host(key)))
        ctx.set_path(0)
        for z, key in got[1:]:
            assert np.array_equal(z, got[0][0]) and key == got[0][1]


@pytest.mark.parametrize("p16", [False, True], ids=["f32", "p16"])
@pytest.mark.parametrize("n_tau", [1, 5, 16, 19])
def test_delay_grid_scorers_at_group_edges(stt, ctx, n_tau, p16):
    T, F = 33, 64
    m = _map(stt, T, F)
    if p16:
        m = ctx.pack_p16(m)
    for n in (1, 5, F, F + 1, 4103):
        _say("delay routes", n_tau, p16, n)
        tr = _tracks(ctx, stt, T, F, n)
        got = []
        for path in (3, 1, 0, 2):
            ctx.set_path(path)
            z, mi, key = ctx.score_maxdelay(m, -DT, DT // 8, n_tau, tracks=tr)
            got.append((*_host(z, mi), key_to_host(key)))
        ctx.set_path(0)
        for z, mi, key in got[1:]:
            assert np.array_equal(z, got[0][0]) and np.array_equal(mi, got[0][1]) and key == got[0][2]


# per (T, F): both sides of the slab threshold (6e7 pixels' worth) and of the one wave / one lane one
# (80000 T / (T + 600) templates)
@pytest.mark.parametrize("T,F,ns", [(20, 200, (2580, 2581, 100_000)), (300, 100, (26_666, 26_667, 199_999, 200_000)),
                                    (1000, 300, (49_999, 50_000, 59_999, 60_000))])
def test_routes_by_size(stt, ctx, T, F, ns):
    m = _map(stt, T, F)
    g = stt.Gen(seed=11, min_len=10, dtau_max=DT)
    for n in ns:
        _say("by size", T, F, n)
        z, key = ctx.score(m, gen=g, n=n, first=5)
        ctx.set_path(1)
        z1, key1 = ctx.score(m, gen=g, n=n, first=5)
        ctx.set_path(0)
        assert np.array_equal(*_host(z, z1)) and key_to_host(key) == key_to_host(key1)


# both sides of the template counts and column widths at which the slab shape changes (4 KB columns
# at F = 512, 12 KB at F = 1536)
@pytest.mark.parametrize("F", [100, 500, 512, 1528, 1536])
def test_slab_shapes_by_size(stt, F):
    T = 24
    c = stt.Context(0)  # of its own: a set shape stays set
    m = _map(stt, T, F)
    g = stt.Gen(seed=12, min_len=10, dtau_max=DT)
    ns = (4096, 399_999, 400_000, 600_000, 1_500_000, 2_000_000)
    c.set_path(2)
    auto = []
    for n in ns:
        _say("shape by size", F, n)
        z, key = c.score(m, gen=g, n=n)
        auto.append((*_host(z), key_to_host(key)))
    c.set_slab_shape(1024, 4)
    for n, (z, key) in zip(ns, auto):
        z4, key4 = c.score(m, gen=g, n=n)
        assert np.array_equal(*_host(z4), z) and key_to_host(key4) == key
    keys = []
    for wg, tpt in ((0, 0), (1024, 4)):
        b = stt.Context(0)
        if wg:
            b.set_slab_shape(wg, tpt)
        k = b.score_batch([m, _map(stt, T, F, seed=6)], g, [300_000, 110_000])
        keys.append(k.cpu().numpy())
        b.close()
    assert np.array_equal(keys[0], keys[1])
    c.close()


# both sides of the rule by which a wave per template gathers from the caller's map or folds it first:
# 250 000 pixels, 1024 columns, n T = 1.2e6
@pytest.mark.parametrize("T,F,n", [(500, 499, 2000), (500, 500, 2000), (500, 500, 2400), (500, 500, 2401),
                                   (1024, 245, 1171), (1024, 245, 1172), (1025, 245, 1000)])
def test_wave_scorers_folded_or_not(stt, ctx, T, F, n):
    m = _map(stt, T, F)
    tr = _tracks(ctx, stt, T, F, n)
    print("folded or not", T, F, n, flush=True, file=sys.stderr)
    got = []
    for path in (3, 1):
        ctx.set_path(path)
        z, key = ctx.score(m, tracks=tr)
        zd, mi, keyd = ctx.score_maxdelay(m, -DT, DT // 8, 9, tracks=tr)
        got.append((_host(z, zd, mi), key_to_host(key), key_to_host(keyd)))
    ctx.set_path(0)
    for a, b in zip(got[0][0], got[1][0]):
        assert np.array_equal(a, b)
    assert got[0][1:] == got[1][1:]


# both sides of the template counts at which the delay grid (T = 100: one wave to one lane per
# template near 7391, slabs from 400 000) and the free-t_mid scorer (slabs from 23 572) change scorers
@pytest.mark.parametrize("n", [7390, 7392, 399_999, 400_000])
def test_delay_grid_routes_by_size(stt, ctx, n):
    m = _map(stt, 100, 64)
    g = stt.Gen(seed=13, min_len=10, dtau_max=DT)
    got = []
    for path in (0, 1, 2):
        print("delay route", n, path, flush=True, file=sys.stderr)
        ctx.set_path(path)
        z, mi, key = ctx.score_maxdelay(m, -DT, DT // 4, 9, gen=g, n=n, first=3)
        got.append((*_host(z, mi), key_to_host(key)))
    ctx.set_path(0)
    for z, mi, key in got[1:]:
        assert np.array_equal(z, got[0][0]) and np.array_equal(mi, got[0][1]) and key == got[0][2]


@pytest.mark.parametrize("p16", [False, True], ids=["f32", "p16"])
@pytest.mark.parametrize("n", [4095, 23_571, 23_572, 60_000])
def test_tmid_routes_by_size(stt, ctx, n, p16):
    m = _map(stt, 100, 64)
    if p16:
        m = ctx.pack_p16(m)
    g = stt.Gen(seed=14, min_len=10, dtau_max=DT)
    got = []
    for path in (0, 2, 3):
        print("t_mid route", n, p16, path, flush=True, file=sys.stderr)
        ctx.set_path(path)
        z, key = ctx.score_tm(m, gen=g, n=n, first=3)
        got.append((*_host(z), key_to_host(key)))
    ctx.set_path(0)
    for z, key in got[1:]:
        assert np.array_equal(z, got[0][0]) and key == got[0][1]


# a lane's gathers one at a time or a flush group's: maps on both sides of 4 MB, templates on both sides of
# 40 000 active lanes, templates that start and end within their groups
@pytest.mark.parametrize("T,F,n", [(100, 5300, 130_000), (100, 5300, 100_000), (33, 4000, 200_000)])
def test_lane_gathers(stt, ctx, T, F, n):
    m = _map(stt, T, F)
    pm = ctx.pack_p16(m)
    g = stt.Gen(seed=15, min_len=3, dtau_max=DT)
    print("lane gathers", T, F, n, flush=True, file=sys.stderr)
    for mm in (m, pm):
        got = []
        for path in (1, 3):
            ctx.set_path(path)
            z, key = ctx.score(mm, gen=g, n=n, first=9)
            zd, mi, keyd = ctx.score_maxdelay(mm, -DT, DT // 8, 9, gen=g, n=n, first=9)
            got.append((_host(z, zd, mi), key_to_host(key), key_to_host(keyd)))
        ctx.set_path(0)
        assert all(np.array_equal(a, b) for a, b in zip(got[0][0], got[1][0])) and got[0][1:] == got[1][1:]
