"""Performance cases of the template search: what a user of the library has it do, over the range of sizes.

A case is a dict of plain values. ``prepare`` makes what a program holds before the call (maps, strain, keys,
template lists, the context), ``run`` is one pass through the public entry points, ``work`` counts the bytes and
flops the pass cannot do without, and ``exact`` evaluates the same definition in FP64 with plain torch.

Kinds:
  list       the given templates scored again on one map (the plain re-score that ends a refinement)
  score      a random search on one map that keeps every template's score and the best key
  argmax     a random search that keeps only the loudest template, read back by the host
  fp16       a map packed to FP16, searched, and the top K re-scored in FP64 on the FP32 map
  batch      many background maps of uneven duration, one best key per map
  tmid       a random search with a free t_mid
  maxdelay   each template maximised over a grid of delays
  refine     a search, its top K, and their projected gradient ascent
  grad       the smooth statistic and its gradient through torch's autograd
  mapform    two detectors' strain to spectra and time-slide maps
  signif     the false-alarm probability of foreground maxima and the threshold of a background
"""
import math

import numpy as np
import torch

import paper_1401_8060_amd.stt as stt
from paper_1401_8060_amd.autograd import smooth_snr

DTAU_MAX = stt.dtau_units(0.010)  # the all-sky delay of 10 ms
UNIT = 2.0 ** -28                 # s
DEV = "cuda"


def listed():
    return [
        # the smallest call: 1024 refined candidates scored again with the plain statistic (latency)
        dict(name="list_1000x1000_1024", kind="list", T=1000, F=1000, n=1024, L=10),
        # a small search: the plain 100 x 128 map with 10^4 templates (latency and launches)
        dict(name="score_100x128_1e4", kind="score", T=100, F=128, n=10_000, L=10, tuned=False),
        # the headline search: 10^7 templates, every score kept, in the tuned shape the benchmark uses
        dict(name="score_1000x1000_1e7", kind="score", T=1000, F=1000, n=10_000_000, L=10, tuned=True),
        # the paper's Table III shape, 2 x 10^7 templates of at least 35 s, the loudest kept
        dict(name="argmax_500x151_2e7", kind="argmax", T=500, F=151, n=20_000_000, L=70, tuned=True),
        # FP16 storage: pack, 2 x 10^7 templates, top 1024, FP64 re-score
        dict(name="fp16_2000x2000_2e7", kind="fp16", T=2000, F=2000, n=20_000_000, L=10, K=1024),
        # the background: 64 maps of 500 to 2000 columns, 10^6 templates each, in one launch
        dict(name="batch_64maps_1e6", kind="batch", maps=64, T_lo=500, T_hi=2000, F=1000, n=1_000_000, L=10),
        # all six random numbers: the free-t_mid search of the headline map
        dict(name="tmid_1000x1000_1e7", kind="tmid", T=1000, F=1000, n=10_000_000, L=10),
        # delay-maximised scores: 16 delays spanning the all-sky band
        dict(name="maxdelay_1000x1000_1e6x16", kind="maxdelay", T=1000, F=1000, n=1_000_000, L=10, n_tau=16),
        # differentiation: a search of 10^6, its top 1024 refined for 50 steps
        dict(name="refine_1000x1000_1e6", kind="refine", T=1000, F=1000, n=1_000_000, L=10, K=1024, steps=50),
        # one forward and backward pass over 1024 templates, as a gradient-based program of its own takes it
        dict(name="grad_1000x1000_1024", kind="grad", T=1000, F=1000, n=1024, L=10),
        # map formation: 500 s of two detectors at 4096 Hz into 256 time-slide maps
        dict(name="mapform_1000x1000_256", kind="mapform", T=1000, F=1000, M=4096, nb=4, slides=256),
        # significance: 1000 foreground maxima against 10^6 background maxima, FAP < 0.1 %
        dict(name="signif_1e3_1e6", kind="signif", n_fg=1000, n_bg=1_000_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["list", "score", "score", "argmax", "fp16", "batch", "tmid", "maxdelay", "refine", "grad", "mapform",
                       "signif"])
    if kind == "signif":
        return dict(kind=kind, n_fg=_log(rng, 1, 20_000), n_bg=_log(rng, 1000, 1_000_000))
    if kind == "mapform":
        M = rng.choice([512, 1024, 2048, 4096, 8192])
        return dict(kind=kind, T=_log(rng, 100, 1500), F=_log(rng, 60, M // 2 - M // 32), M=M, nb=rng.choice([2, 4, 8]),
                    slides=_log(rng, 1, 128))
    T, F = _log(rng, 100, 2000), _log(rng, 100, 2000)
    L = rng.choice([10, max(2, T // 8)])
    if kind == "list":
        return dict(kind=kind, T=T, F=F, n=_log(rng, 100, 3000), L=L)
    if kind in ("score", "argmax"):
        return dict(kind=kind, T=T, F=F, n=_log(rng, 1000, 10_000_000), L=L, tuned=False)
    if kind == "fp16":
        n = _log(rng, 10_000, 20_000_000)
        return dict(kind=kind, T=T, F=F, n=n, L=L, K=_log(rng, 16, 2048))
    if kind == "batch":
        lo = min(T, 1000)
        return dict(kind=kind, maps=_log(rng, 2, 64), T_lo=lo, T_hi=2 * lo, F=min(F, 1200), n=_log(rng, 10_000, 1_000_000),
                    L=10)
    if kind == "tmid":
        return dict(kind=kind, T=T, F=F, n=_log(rng, 1000, 5_000_000), L=L)
    if kind == "maxdelay":
        return dict(kind=kind, T=T, F=F, n=_log(rng, 1000, 500_000), L=L, n_tau=rng.randint(2, 32))
    if kind == "refine":
        return dict(kind=kind, T=T, F=F, n=_log(rng, 20_000, 1_000_000), L=L, K=_log(rng, 16, 1024), steps=rng.choice([20, 50]))
    return dict(kind="grad", T=T, F=F, n=_log(rng, 64, 4096), L=L)


# ------------------------------------------------------------------------------------------------ inputs

def _rng(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(1_000_003 * seed + 7919 * salt + 17)


def _noise_map(T, F, seed, salt=0, inject=True):
    """Gaussian noise Y = sigma (n + i n') with log-uniform sigma on [0.5, 2], one quadratic track at SNR 8."""
    g = _rng(seed, salt)
    s = torch.exp(math.log(0.5) + math.log(4.0) * torch.rand((T, F), generator=g, device=DEV))
    Y = torch.view_as_complex(torch.randn((T, F, 2), generator=g, device=DEV) * s[..., None])
    if inject:
        N = max(2, int(0.6 * T))
        t = torch.arange(N, device=DEV) + T // 5
        x = torch.arange(N, device=DEV, dtype=torch.float64) / (N - 1)
        r = (F * ((1 - x) ** 2 * 0.25 + 2 * (1 - x) * x * 0.6 + x ** 2 * 0.45)).floor().long()
        ph = -2 * math.pi * (100.0 + r) * 0.003
        Y[t, r] += (s[t, r] * (8.0 / math.sqrt(N)) * torch.exp(1j * ph)).to(Y.dtype)
    return stt.Map(Y, s)


def _gen(c, seed):
    return stt.Gen(seed=seed + 1, stream=0, min_len=c["L"], dtau_max=DTAU_MAX)


def _theta(c, seed, n):
    """Continuous templates, as the iterates of an ascent: no coordinate on the grid's nodes."""
    T, F = c["T"], c["F"]
    g = _rng(seed, 3)
    u = torch.rand((n, 6), generator=g, device=DEV)
    span = (0.1 + 0.6 * u[:, 1]) * (T - 1)
    t0 = u[:, 0] * (T - 1 - span)
    ph = 0.5 + u[:, 2:5] * (F - 2)
    th = torch.cat([t0[:, None], (t0 + span)[:, None], ph, (20.0 * u[:, 5:6] - 10.0)], 1).contiguous()
    K = (span.floor() + 1).to(torch.int32).clamp(min=2).contiguous()
    return th, K


def _batch_T(c, seed):
    u = np.random.default_rng(seed + 5).random(c["maps"])
    return [int(c["T_lo"] + math.floor(x * (c["T_hi"] - c["T_lo"] + 1))) for x in u]


def _spectro(c):
    # columns of 1 s (fs = M); the band starts at a tenth of it, at most where F bins still fit below M/2
    return stt.Spectro(fs=float(c["M"]), M=c["M"], k_lo=min(100, c["M"] // 2 - c["F"]), F=c["F"], nb=c["nb"])


def _strain(c, seed):
    n = (c["T"] + 1) * c["M"] // 2
    g = _rng(seed, 11)
    t = torch.arange(n, device=DEV, dtype=torch.float64) / c["M"]
    out = []
    for k in range(2):
        x = torch.randn(n, generator=g, device=DEV, dtype=torch.float32)
        u = t - 0.003 * k  # a chirp that reaches the second detector 3 ms later
        f0 = 0.06 * c["M"]
        out.append((x + 0.02 * torch.cos(2 * math.pi * (f0 * u + 0.5 * u * u)).float()).contiguous())
    return out


def _keys(n, seed, salt):
    """Best keys of n maps: scores like the maxima of many N(0, 1) (a Gumbel law), random template indices."""
    g = _rng(seed, salt)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64).clamp(1e-12, 1 - 1e-12)
    z = (5.0 - 0.2 * torch.log(-torch.log(u))).float()
    j = torch.randint(0, 1_000_000, (n,), generator=g, device=DEV)
    o = z.view(torch.int32).long() + 2 ** 31  # positive scores: the sign bit set
    return ((o - 2 ** 32) << 32) + (0xFFFFFFFF - j), z


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    ctx = stt.Context(0)
    st = dict(c=c, ctx=ctx, kind=kind)
    if kind == "signif":
        st["bg"], _ = _keys(c["n_bg"], seed, 1)
        st["fg"], _ = _keys(c["n_fg"], seed, 2)
        return st
    if kind == "mapform":
        T, F, ns = c["T"], c["F"], c["slides"]
        st["p"], st["x"] = _spectro(c), _strain(c, seed)
        st["shifts"] = [2 * k for k in range(ns)]
        st["spec"] = [torch.empty((T, F), dtype=torch.complex64, device=DEV) for _ in range(2)]
        st["psd"] = [torch.empty((T, F), dtype=torch.float32, device=DEV) for _ in range(2)]
        st["Y"] = torch.empty((ns, T, F), dtype=torch.complex64, device=DEV)
        st["sigma"] = torch.empty((ns, T, F), dtype=torch.float32, device=DEV)
        lo, d = st["p"].fq4()
        st["maps"] = [stt.Map(st["Y"][k], st["sigma"][k], lo, d) for k in range(ns)]
        return st
    if kind == "batch":
        st["maps"] = [_noise_map(T, c["F"], seed, k, inject=False) for k, T in enumerate(_batch_T(c, seed))]
        st["g"], st["n"] = _gen(c, seed), [c["n"]] * c["maps"]
        st["keys"] = torch.zeros(c["maps"], dtype=torch.int64, device=DEV)
        return st
    m = st["m"] = _noise_map(c["T"], c["F"], seed)
    g = st["g"] = _gen(c, seed)
    n = c["n"]
    if kind == "list":
        st["tracks"] = ctx.make_tracks(g, c["T"], c["F"], 0, n)
    if kind == "grad":
        st["theta"], st["K"] = _theta(c, seed, n)
        st["theta"].requires_grad_(True)
        st["gz"] = torch.rand(n, generator=_rng(seed, 4), device=DEV) + 0.5
        return st
    if c.get("tuned"):
        import os
        ctx.autotune(m, g, n, os.path.join(os.path.dirname(stt.__file__), "tuning", "gfx950.json"))
    if kind != "argmax":
        st["snr"] = torch.empty(n, dtype=torch.float32, device=DEV)
    if kind == "maxdelay":
        st["tidx"] = torch.empty(n, dtype=torch.int32, device=DEV)
        st["d0"], st["step"] = -DTAU_MAX, 2 * DTAU_MAX // (c["n_tau"] - 1)
    if kind == "score":
        st["key"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return st


def run(st):
    c, ctx, kind = st["c"], st["ctx"], st["kind"]
    if kind == "list":
        snr, _ = ctx.score(st["m"], tracks=st["tracks"], snr=st["snr"])
        return snr
    if kind == "score":
        st["key"].zero_()
        snr, key = ctx.score(st["m"], gen=st["g"], n=c["n"], snr=st["snr"], best_key=st["key"])
        return dict(snr=snr, key=key)
    if kind == "argmax":
        _, key = ctx.score(st["m"], gen=st["g"], n=c["n"], snr=None)
        z, j = stt.decode_best(key)
        return dict(z=z, j=j)
    if kind == "fp16":
        pm = ctx.pack_p16(st["m"])
        snr, _ = ctx.score(pm, gen=st["g"], n=c["n"], snr=st["snr"])
        idx, val = ctx.topk(snr, c["K"])
        return dict(packed=pm.data, scale_exp=pm.scale_exp, snr=snr, idx=idx, val=val,
                    z64=ctx.rescore_f64(st["m"], idx, gen=st["g"]))
    if kind == "batch":
        st["keys"].zero_()
        return ctx.score_batch(st["maps"], st["g"], st["n"], best_keys=st["keys"])
    if kind == "tmid":
        snr, key = ctx.score_tm(st["m"], gen=st["g"], n=c["n"], snr=st["snr"])
        return dict(snr=snr, key=key)
    if kind == "maxdelay":
        snr, tidx, _ = ctx.score_maxdelay(st["m"], st["d0"], st["step"], c["n_tau"], gen=st["g"], n=c["n"], snr=st["snr"],
                                          tau_idx=st["tidx"])
        return dict(snr=snr, tau_idx=tidx)
    if kind == "refine":
        snr, _ = ctx.score(st["m"], gen=st["g"], n=c["n"], snr=st["snr"])
        idx, val = ctx.topk(snr, c["K"])
        theta, K = ctx.tracks_to_theta(ctx.tracks_at(st["g"], c["T"], c["F"], idx))
        th, zs, tracks, zp = ctx.refine(st["m"], theta, K, c["L"], DTAU_MAX, steps=c["steps"])
        return dict(snr=snr, idx=idx, val=val, theta=th, z_smooth=zs, tracks=tracks, z_plain=zp)
    if kind == "grad":
        z = smooth_snr(ctx, st["m"], st["theta"], st["K"])
        (grad,) = torch.autograd.grad(z, st["theta"], st["gz"])
        return dict(z=z, grad=grad)
    if kind == "mapform":
        p, T = st["p"], c["T"]
        for k in range(2):
            ctx.spectra(st["x"][k], p, T, st["spec"][k], st["psd"][k])
        ctx.form_maps(p, st["spec"][0], st["psd"][0], st["spec"][1], st["psd"][1], st["shifts"], out=st["maps"])
        return dict(spec_i=st["spec"][0], spec_j=st["spec"][1], psd_i=st["psd"][0], psd_j=st["psd"][1], Y=st["Y"],
                    sigma=st["sigma"])
    cnt, fap, za = ctx.significance(st["bg"], st["fg"], alpha=1e-3)
    return dict(n_louder=cnt, fap=fap, z_alpha=za)


def work(case):
    c = case
    kind = c["kind"]
    if kind == "signif":
        # each key read once, each output written once; ranking n_fg values in a sorted background
        n = c["n_fg"] + c["n_bg"]
        return dict(bytes=8 * n + 12 * c["n_fg"] + 4, flops=n * math.log2(max(2, c["n_bg"])))
    if kind == "mapform":
        px, n = c["T"] * c["F"], (c["T"] + 1) * c["M"] // 2
        return dict(bytes=2 * 4 * n + 2 * 12 * px + 12 * px * c["slides"],
                    flops=2 * c["T"] * 2.5 * c["M"] * math.log2(c["M"]) + 2 * px * 4 + 9 * px * c["slides"])
    if kind == "grad":
        K = 0.4 * (c["T"] - 1) * c["n"]  # mean samples; 4 nodes each for the value, and again for the gradient
        return dict(bytes=12 * c["T"] * c["F"] + c["n"] * 80, flops=K * (4 * 11 + 4 * 16 + 30))
    T = (c["T_lo"] + c["T_hi"]) / 2 if kind == "batch" else c["T"]
    maps = c.get("maps", 1)
    px = c["n"] * maps * (c["L"] + (T - c["L"]) / 3.0)  # mean length of the pairs (t0, t2)
    bytes_ = 12 * T * c["F"] * maps
    flops = 8.0 * px * c.get("n_tau", 1)
    if kind == "list":
        bytes_ += 28 * c["n"]
    elif kind in ("score", "tmid", "refine"):
        bytes_ += 4 * c["n"]
    elif kind == "fp16":
        bytes_ += 4 * T * c["F"] + 4 * c["n"]
    elif kind == "maxdelay":
        bytes_ += 8 * c["n"]
    if kind == "refine":
        flops += (c["steps"] + 1) * c["K"] * (c["L"] + (T - c["L"]) / 3.0) * (4 * 16 + 30)
    return dict(bytes=bytes_, flops=flops)


# ------------------------------------------------------------------------------------------------ FP64 definition

_M32 = 0xFFFFFFFF


def _philox(seed, n, block, stream=0):
    """Words of Philox4x32-10 at counters (j, 0, stream, block), j < n, key = seed, as int64 tensors."""
    x = torch.arange(n, device=DEV, dtype=torch.int64)
    c = [x, torch.zeros_like(x), torch.full_like(x, stream), torch.full_like(x, block)]
    k0, k1 = seed & _M32, (seed >> 32) & _M32

    def mul(a, b):  # 32 x 32 -> (high, low) without overflowing int64
        lo, hi = a * (b & 0xFFFF), a * (b >> 16)
        t = (lo >> 16) + hi
        return (t >> 16) & _M32, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)

    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
    return c


def _scale(hi, lo, m):
    """floor((hi 2^32 + lo) m / 2^64) for m < 2^31."""
    return (hi * m + ((lo * m) >> 32)) >> 32


def _templates(c, seed):
    T, F, L, n = c["T"], c["F"], c["L"], c["n"]
    a, b = _philox(seed + 1, n, 0), _philox(seed + 1, n, 1)
    npos = T - L + 1
    k = _scale(a[0], a[1], npos * (npos + 1) // 2)
    e = ((torch.sqrt(8.0 * k.double() + 1.0) - 1.0) / 2.0).long()
    e = e - (e * (e + 1) // 2 > k).long()
    e = e + ((e + 1) * (e + 2) // 2 <= k).long()
    t0 = k - e * (e + 1) // 2
    t2 = e + L - 1
    f = [(w * (F << 8)) >> 32 for w in (a[2], a[3], b[0])]
    dtau = _scale(b[1], b[2], 2 * DTAU_MAX + 1) - DTAU_MAX
    t1 = t0 + ((b[3] * (t2 - t0 + 1)) >> 32)
    return dict(t0=t0, t1=t1, t2=t2, f0=f[0], f1=f[1], f2=f[2], dtau=dtau)


def _rows_plain(tr, k):
    Dt = (tr["t2"] - tr["t0"])[:, None]
    num = (Dt - k) ** 2 * tr["f0"][:, None] + 2 * (Dt - k) * k * tr["f1"][:, None] + k * k * tr["f2"][:, None]
    return torch.div(num, Dt * Dt * 256, rounding_mode="floor")


def _row_tm_exact(t0, t1, t2, f0, f1, f2, dt):
    """The row of one free-t_mid pixel in integers."""
    a, b = t0 - 2 * t1 + t2, 2 * (t1 - t0)
    B, C = 2 * (f1 - f0), f0 - 2 * f1 + f2
    if a == 0:
        Dt = t2 - t0
        return (Dt * Dt * f0 + B * Dt * dt + C * dt * dt) // (256 * Dt * Dt)
    D = b * b + 4 * a * dt
    V, W = a * B - C * b, 512 * a * a  # f/256 = (U + V sqrt(D)) / W, W > 0
    U = 2 * a * a * f0 - b * V + 2 * a * C * dt

    def at_least(r):  # U + V sqrt(D) >= r W
        x = r * W - U
        if V >= 0:
            return x <= 0 or V * V * D >= x * x
        return x <= 0 and V * V * D <= x * x

    r = (U + (1 if V >= 0 else -1) * math.isqrt(V * V * D)) // W
    while at_least(r + 1):
        r += 1
    while not at_least(r):
        r -= 1
    return r


def _rows_tm(tr, k):
    col = {q: v[:, None] for q, v in tr.items()}
    a, b = (col["t0"] - 2 * col["t1"] + col["t2"]).double(), (2 * (col["t1"] - col["t0"])).double()
    B, C = (2 * (col["f1"] - col["f0"])).double(), (col["f0"] - 2 * col["f1"] + col["f2"]).double()
    kd = k.double()
    den = b + torch.sqrt((b * b + 4 * a * kd).clamp(min=0))
    xi = torch.where(k > 0, 2 * kd / den, torch.zeros_like(den))
    y = (col["f0"].double() + xi * (B + C * xi)) / 256.0
    row = y.floor().long()
    near = ((y - y.round()).abs() < 1e-7) & (k <= col["t2"] - col["t0"])
    i, j = near.nonzero(as_tuple=True)
    if i.numel():
        rec = torch.stack([tr[q][i] for q in ("t0", "t1", "t2", "f0", "f1", "f2")] + [k.expand_as(row)[i, j]], 1).tolist()
        row[i, j] = torch.tensor([_row_tm_exact(*r) for r in rec], device=DEV)
    return row


def _scores(m, tr, rows_of, delays=None):
    """z of every template in FP64 (S / sqrt(N)), or its maximum over the given delays."""
    p = (m.Y.to(torch.complex128) / m.sigma.double()).reshape(-1)
    n = tr["t0"].numel()
    N = tr["t2"] - tr["t0"] + 1
    out = torch.empty(n, dtype=torch.float64, device=DEV)
    order = torch.argsort(N)
    sizes = N[order].cpu().numpy()
    a = 0
    while a < n:
        b = min(n, a + max(1, int(2e7 // sizes[min(n - 1, a)])))
        b = max(a + 1, min(b, a + max(1, int(2e7 // sizes[b - 1]))))
        s = order[a:b]
        t = {q: v[s] for q, v in tr.items()}
        k = torch.arange(int(sizes[b - 1]), device=DEV)[None]
        on = k < N[s][:, None]
        row = rows_of(t, k).clamp(0, m.F - 1)
        px = torch.where(on, p[((t["t0"][:, None] + k).clamp(max=m.T - 1) * m.F + row)], torch.zeros((), dtype=p.dtype, device=DEV))
        f = 2 * math.pi * UNIT * (100.0 + row)
        if delays is None:
            ph = f * t["dtau"][:, None]
            S = (torch.cos(ph) * px.real - torch.sin(ph) * px.imag).sum(1)
        else:
            S = torch.stack([(torch.cos(f * d) * px.real - torch.sin(f * d) * px.imag).sum(1) for d in delays], 1).max(1)[0]
        out[s] = S / torch.sqrt(N[s].double())
        a = b
    return out


def _smooth(m, theta, K, gz):
    p = m.Y.to(torch.complex128) / m.sigma.double()
    T, F = m.T, m.F
    z, grad = [], []
    for a in range(0, theta.shape[0], 256):
        th, Kk = theta[a:a + 256].double(), K[a:a + 256].long()
        k = torch.arange(int(Kk.max()), device=DEV)[None].double()
        on = (k < Kk[:, None]).double()
        xi = k / (Kk[:, None] - 1).double()
        w = [(1 - xi) ** 2, 2 * xi * (1 - xi), xi ** 2]
        u0 = th[:, :1] + xi * (th[:, 1:2] - th[:, :1])
        v0 = sum(w[q] * th[:, 2 + q:3 + q] for q in range(3)) - 0.5
        u, v = u0.clamp(0, T - 1), v0.clamp(0, F - 1)
        ut, vt = ((u0 >= 0) & (u0 <= T - 1)).double() * on, ((v0 >= 0) & (v0 <= F - 1)).double() * on
        i, r = u.floor().long().clamp(max=T - 2), v.floor().long().clamp(max=F - 2)
        A, B = u - i, v - r
        G, D = {}, {}
        for x in (0, 1):
            for y in (0, 1):
                q = p[i + x, r + y]
                f = 2 * math.pi * (100.0 + r + y)
                ph = f * th[:, 5:6] * 1e-3
                G[x, y] = torch.cos(ph) * q.real - torch.sin(ph) * q.imag
                D[x, y] = -f * (torch.sin(ph) * q.real + torch.cos(ph) * q.imag) * 1e-3
        W = {(0, 0): (1 - A) * (1 - B), (1, 0): A * (1 - B), (0, 1): (1 - A) * B, (1, 1): A * B}
        du = ut * ((1 - B) * (G[1, 0] - G[0, 0]) + B * (G[1, 1] - G[0, 1]))
        dv = vt * ((1 - A) * (G[0, 1] - G[0, 0]) + A * (G[1, 1] - G[1, 0]))
        sc = Kk.double() ** -0.5
        z.append((on * sum(W[q] * G[q] for q in W)).sum(1) * sc)
        cols = [((1 - xi) * du).sum(1), (xi * du).sum(1)] + [(w[q] * dv).sum(1) for q in range(3)]
        cols.append((on * sum(W[q] * D[q] for q in W)).sum(1))
        grad.append(torch.stack(cols, 1) * sc[:, None])
    return torch.cat(z), torch.cat(grad) * gz.double()[:, None]


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "signif":
        bg, fg = (_keys(c[k], seed, s)[1].double() for k, s in (("n_bg", 1), ("n_fg", 2)))
        srt = bg.sort()[0]
        louder = c["n_bg"] - torch.searchsorted(srt, fg, side="left")
        m = max(1, math.ceil(1e-3 * c["n_bg"]))
        return dict(n_louder=None, fap=louder.double() / c["n_bg"], z_alpha=srt[-m].reshape(1))
    if kind == "mapform":
        T, F, M, nb = c["T"], c["F"], c["M"], c["nb"]
        lo = _spectro(c).k_lo
        win = torch.sin(math.pi * torch.arange(M, device=DEV, dtype=torch.float64) / M) ** 2
        scale = 2.0 / (M / float(M) * 0.375)
        spec, psd = [], []
        for x in _strain(c, seed):
            seg = x.double().unfold(0, M, M // 2)[:T] * win
            s = torch.fft.rfft(seg, dim=1)[:, lo:lo + F] / float(M)
            pw = scale * s.abs() ** 2
            acc, cnt = torch.zeros_like(pw), torch.zeros((T, 1), dtype=torch.float64, device=DEV)
            for d in range(2, nb + 2):
                acc[d:] += pw[:-d]
                cnt[d:] += 1
                acc[:-d] += pw[d:]
                cnt[:-d] += 1
            spec.append(s)
            psd.append(acc / cnt)
        ns = c["slides"]
        Y = torch.empty((ns, T, F), dtype=torch.complex128, device=DEV)
        sg = torch.empty((ns, T, F), dtype=torch.float64, device=DEV)
        for k in range(ns):
            Y[k] = scale * spec[0].conj() * spec[1].roll(-2 * k, 0)
            sg[k] = torch.sqrt(0.5 * psd[0] * psd[1].roll(-2 * k, 0))
        return dict(spec_i=spec[0], spec_j=spec[1], psd_i=psd[0], psd_j=psd[1], Y=Y, sigma=sg)
    if kind in ("batch", "refine"):
        return None  # packed keys; the end of an ascent of many rounded steps
    m = _noise_map(c["T"], c["F"], seed)
    if kind == "grad":
        th, K = _theta(c, seed, c["n"])
        gz = torch.rand(c["n"], generator=_rng(seed, 4), device=DEV) + 0.5
        z, grad = _smooth(m, th, K, gz)
        return dict(z=z, grad=grad)
    tr = _templates(c, seed)
    if kind == "list":
        return _scores(m, tr, _rows_plain)
    if kind == "score":
        return dict(snr=_scores(m, tr, _rows_plain), key=None)
    if kind == "argmax":
        return dict(z=float(_scores(m, tr, _rows_plain).max()), j=None)
    if kind == "fp16":
        return dict(packed=None, scale_exp=None, snr=_scores(m, tr, _rows_plain), idx=None, val=None, z64=None)
    if kind == "tmid":
        return dict(snr=_scores(m, tr, _rows_tm), key=None)
    d0, step = -DTAU_MAX, 2 * DTAU_MAX // (c["n_tau"] - 1)
    return dict(snr=_scores(m, tr, _rows_plain, [float(d0 + q * step) for q in range(c["n_tau"])]), tau_idx=None)
