"""Workloads that the library's speed is measured on.

Every case is one call (or one replayed step) through the public entry points
on inputs that are already on the GPU, as a detrending program or the serving
loop makes it: single curves, packed batches of equal or ragged curves, the
options a study of the method uses, and a plan's step over a resident arena.

listed()  the named cases; draw(rng)  one more from the same ranges;
prepare(case, seed)  inputs from the seed, and the plan where one is kept;
run(state)  one pass; work(case)  the bytes and operations of a pass;
exact(case, seed)  the outputs in 64 bits, by plain torch.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2604_06602_amd as umi

MIN = 1.0 / 1440.0
TESS_DT = 2 * MIN          # TESS two-minute cadence
KEPLER_DT = 29.4 * MIN     # Kepler long cadence
GAP_DAYS = 0.5             # a longer step between valid samples ends a segment

# What a case may leave out.  `n` is the length of every curve, or `n` .. `n_hi`
# the range ragged curves are drawn from (uniformly, or over the logarithm);
# `W` one window, or 0 for one of 25, 121, 361 and 721 per curve.
DEFAULTS = dict(kind="batch", curves=1, n=20000, n_hi=0, log=False, W=361, cadence="tess",
                gaps="none", time=True, median=False, detrended=False, alpha=2.0, c=5.0, iters=5,
                presets=False, scale="upper_rms", window_days=0.0, sigma=1e-3, shape_seed=1)
MIXED_W = (25, 121, 361, 721)
PRESETS = ((2.0, 5.0), (3.0, 5.0), (1.0, 5.0), (10.0, 2.5))  # (alpha, c) by use


def listed():
    return [
        # the smallest call: one short Kepler-cadence curve, all latency
        dict(name="one_1k_w25", kind="one", n=1000, W=25, cadence="kepler"),
        # one TESS curve with its median, as the smoke check and an interactive user call it
        dict(name="one_20k_w361", kind="one", n=20000, W=361, median=True),
        # one gappy curve of odd length without a time array and with a wide window
        dict(name="one_odd_9337_w721", kind="one", n=9337, W=721, gaps="random", time=False),
        # a few curves at once: too small a batch to fill the chip
        dict(name="few_16x20k_w361", curves=16, n=20000, W=361),
        # the headline: a TESS sector's worth of curves with the mid-sector gap
        dict(name="tess_1000x18k_w361", curves=1000, n=18000, W=361, gaps="mid"),
        # Kepler-like ragged curves, the 0.5-day window at long cadence
        dict(name="kepler_2000x40k_70k_w25", curves=2000, n=40000, n_hi=70000, W=25,
             cadence="kepler"),
        # a mixed archive: lengths over two decades, four windows, gaps, use-case settings
        dict(name="mixed_2000x1k_120k", curves=2000, n=1000, n_hi=120000, log=True, W=0,
             gaps="random", presets=True),
        # 27-day stars at the 1.5-day window that long transits need
        dict(name="long_window_200x19440_w1081", curves=200, n=19440, W=1081, gaps="mid"),
        # injection-recovery: the aggressive setting, with the detrended flux
        dict(name="inject_400x19440_w361", curves=400, n=19440, W=361, gaps="mid", alpha=10.0,
             c=2.5, detrended=True),
        # an ablation over irregular cadence: MAD scale, windows given in days
        dict(name="mad_days_100x4408_w121", curves=100, n=4408, W=121, cadence="irregular",
             gaps="random", scale="mad", window_days=0.15, alpha=1.0),
        # one step of the serving loop: a plan replayed over resident mixed curves
        dict(name="plan_step_6_mixed", kind="plan", curves=6, n=1000, n_hi=120000, log=True, W=0,
             gaps="random"),
        # the call for programs that may not allocate, at a four-hour window
        dict(name="noalloc_200x18k_w121", kind="noalloc", curves=200, n=18000, W=121, gaps="mid",
             median=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_COST = 3e11  # lane operations of a drawn case; the largest listed one takes more


def draw(rng):
    """A case of the listed ones' ranges: every kind of call, sizes over their
    logarithm, odd ones included, no dearer than the largest listed case."""
    while True:
        kind = rng.choice(["one", "one", "batch", "batch", "batch", "ragged", "ragged", "options",
                           "plan", "noalloc"])
        c = dict(sigma=round(math.exp(rng.uniform(math.log(5e-5), math.log(2e-3))), 7),
                 gaps=rng.choice(["none", "mid", "random"]), shape_seed=rng.randrange(1 << 20))
        c["W"] = rng.choice([25, 25, 121, 361, 361, 721, 2 * _log_int(rng, 3, 700) + 1])
        c["cadence"] = "kepler" if c["W"] <= 31 else "tess"
        c["alpha"], c["c"] = rng.choice([(2.0, 5.0), (2.0, 5.0), *PRESETS])
        if kind == "one":
            c.update(kind="one", n=_log_int(rng, 1000, 120000), median=rng.random() < 0.5,
                     time=rng.random() < 0.8)
        elif kind in ("batch", "noalloc"):
            c.update(kind=kind, curves=_log_int(rng, 2, 1000), n=_log_int(rng, 1000, 60000),
                     median=rng.random() < 0.5)
            if kind == "noalloc" and c["curves"] * c["n"] > 16_000_000:
                continue
        elif kind == "ragged":
            c.update(curves=_log_int(rng, 8, 2000), n=1000, n_hi=_log_int(rng, 5000, 120000),
                     log=True, presets=rng.random() < 0.5)
            if rng.random() < 0.7:
                c["W"] = 0
        elif kind == "options":
            c.update(curves=_log_int(rng, 4, 200), n=_log_int(rng, 1000, 20000),
                     W=rng.choice([25, 61, 121, 361]), detrended=True,
                     scale=rng.choice(["upper_rms", "mad"]), cadence="irregular")
            if rng.random() < 0.5:
                c["window_days"] = round(c["W"] * TESS_DT * rng.uniform(0.4, 0.9), 4)
        else:
            c.update(kind="plan", curves=_log_int(rng, 1, 40), n=1000, n_hi=120000, log=True, W=0)
        d = _full(c)
        lens, Ws = _shapes(d)
        if sum(n * (33 * w + 2500 * (d["scale"] == "mad") + 500) for n, w in zip(lens, Ws)) \
                <= MOST_COST:
            return c


def _full(case):
    return {**DEFAULTS, **case}


def _shapes(d):
    """Lengths and windows of the case's curves."""
    r = random.Random(d["shape_seed"])
    lens, Ws = [], []
    for _ in range(d["curves"]):
        if not d["n_hi"]:
            lens.append(d["n"])
        elif d["log"]:
            lens.append(_log_int(r, d["n"], d["n_hi"]))
        else:
            lens.append(r.randint(d["n"], d["n_hi"]))
        Ws.append(d["W"] or r.choice(MIXED_W))
    return lens, Ws


def _params(d):
    """alpha and c of the call: one pair, or one of the use-case pairs per curve."""
    if not d["presets"]:
        return d["alpha"], d["c"]
    r = random.Random(d["shape_seed"] + 1)
    p = [PRESETS[min(3, r.randrange(6))] if r.random() < 0.5 else PRESETS[0]
         for _ in range(d["curves"])]
    return (np.array([a for a, _ in p], np.float32), np.array([c for _, c in p], np.float32))


def _curves(d, seed):
    """Packed flux (float32) and time (float64) on the GPU: level 1 with slow
    variability (sinusoids, or correlated noise at Kepler cadence), white
    noise, periodic box transits, flares, and invalid samples."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(int(seed) * 2 + 1)
    lens_list, _ = _shapes(d)
    B, n = len(lens_list), sum(lens_list)
    lens = torch.tensor(lens_list, device=dev)
    off = torch.cumsum(lens, 0) - lens
    cid = torch.repeat_interleave(torch.arange(B, device=dev), lens, output_size=n)
    local = torch.arange(n, device=dev) - off[cid]
    dt = KEPLER_DT if d["cadence"] == "kepler" else TESS_DT

    def u(lo, hi, k=B):
        return lo + (hi - lo) * torch.rand(k, device=dev, generator=g, dtype=torch.float64)

    t = local.double() * dt
    if d["cadence"] == "irregular":
        t = t + 0.4 * dt * (torch.rand(n, device=dev, generator=g, dtype=torch.float64) - 0.5)
    x = 1.0 + d["sigma"] * torch.randn(n, device=dev, generator=g).double()
    if d["cadence"] == "kepler":
        phi = math.exp(-dt / 2.0)  # AR(1), two-day correlation time, std 1e-3
        red = 1e-3 * math.sqrt(1 - phi * phi) * torch.randn(n, device=dev, generator=g)
        step = 1
        while step < 1024:
            red[step:] += phi ** step * red[:-step].clone()
            step *= 2
        x += red
        del red
    else:
        for _ in range(3):
            p, ph = u(1.0, 5.0), u(0.0, 2 * math.pi)
            x += 1e-3 * torch.sin(2 * math.pi * t / p[cid] + ph[cid])
        for _ in range(5):
            lag = t - (u(0.0, 1.0) * lens.double() * dt)[cid]
            x += torch.where(lag >= 0, 5e-3 * torch.exp(-lag.clamp(min=0) / (10 * MIN)), 0.0)
            del lag
    depth, dur = torch.exp(u(math.log(1e-4), math.log(2e-2))), u(1.0, 8.0) / 24.0
    period, epoch = u(1.0, 13.0), u(0.0, 1.0)
    x -= torch.where(torch.remainder(t - (epoch * period)[cid], period[cid]) < dur[cid],
                     depth[cid], 0.0)
    if d["gaps"] == "mid":      # a day without data in the middle of the curve
        half = min(int(0.5 / dt), d["n"] // 8)
        x[(local - (lens // 2)[cid]).abs() < half] = math.nan
    elif d["gaps"] == "random":  # about 5 % of the samples, in gaps of 1 to 48 hours
        mean = 24.5 / 24.0 / dt
        k = max(1, int(0.05 * n / mean))
        at = (u(0.0, 1.0, k) * n).long().clamp(max=n - 1)
        length = (u(1.0, 48.0, k) / 24.0 / dt).long().clamp(min=1)
        end = torch.minimum(at + length, (off + lens)[cid[at]])
        mark = torch.zeros(n + 1, device=dev, dtype=torch.int32)
        one = torch.ones(k, device=dev, dtype=torch.int32)
        mark.index_add_(0, at, one)
        mark.index_add_(0, end, -one)
        x[torch.cumsum(mark, 0)[:n] > 0] = math.nan
    return x.float(), t


class _State:
    pass


def prepare(case, seed):
    d = _full(case)
    s = _State()
    s.d = d
    s.flux, s.time = _curves(d, seed)
    if not d["time"]:
        s.time = None
    lens, Ws = _shapes(d)
    s.lengths = np.array(lens, np.int64)
    s.W = np.array(Ws, np.int32)
    s.alpha, s.c = _params(d)
    s.kw = {}
    if d["scale"] != "upper_rms":
        s.kw["scale"] = d["scale"]
    if d["window_days"] > 0:
        s.kw["window_days"] = d["window_days"]
    if d["kind"] in ("plan", "noalloc"):
        s.trend = torch.empty_like(s.flux)
        s.median = torch.empty_like(s.flux) if d["median"] else None
    if d["kind"] == "plan":
        s.offsets = np.concatenate([[0], np.cumsum(s.lengths)[:-1]]).astype(np.int64)
        s.stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        s.plan = umi.Plan(s.flux, s.time, s.trend, s.median, max_curves=64, max_W=721,
                          stream=s.stream)
    return s


def run(s):
    d = s.d
    if d["kind"] == "one":
        trend, median = umi.detrend(s.flux, s.time, d["W"], s.alpha, s.c, d["iters"], d["median"])
        return _outputs(trend, median, None)
    if d["kind"] == "plan":
        s.plan.run(s.offsets, s.lengths, s.W, s.alpha, s.c, d["iters"])
        return _outputs(s.trend, s.median, None)
    if d["kind"] == "noalloc":
        umi.detrend_batch_noalloc_into(s.flux, s.time, s.lengths, s.W, s.trend, s.median, s.alpha,
                                       s.c, d["iters"])
        return _outputs(s.trend, s.median, None)
    out = umi.detrend_batch(s.flux, s.time, s.lengths, s.W, s.alpha, s.c, d["iters"],
                            with_median=d["median"], with_detrended=d["detrended"], **s.kw)
    return _outputs(out[0], out[1], out[2] if d["detrended"] else None)


def _outputs(trend, median, detrended):
    out = {"trend": trend}
    if median is not None:
        out["median"] = median
    if detrended is not None:
        out["detrended"] = detrended
    return out


def work(case):
    """Flux and times read once, every output written once; the scale and the
    re-weighting iterations summed sample by sample over full windows (3
    operations per sample for the scale, 8 per iteration; selection of the
    medians not counted)."""
    d = _full(case)
    lens, Ws = _shapes(d)
    n = sum(lens)
    per = 4 + (8 if d["time"] else 0) + 4 + (4 if d["median"] else 0) + (4 if d["detrended"] else 0)
    pairs = sum(ln * min(w, ln) for ln, w in zip(lens, Ws))
    return {"bytes": float(n * per), "flops": float(pairs * (3 + 8 * d["iters"]))}


MOST_EXACT = 3e10  # window samples whose 64-bit evaluation takes some ten seconds


def exact(case, seed):
    d = _full(case)
    lens, Ws = _shapes(d)
    if sum(n * w for n, w in zip(lens, Ws)) > MOST_EXACT:
        return None
    flux, time = _curves(d, seed)
    dev = flux.device
    n = flux.numel()
    lens_t = torch.tensor(lens, device=dev)
    cid = torch.repeat_interleave(torch.arange(len(lens), device=dev), lens_t, output_size=n)
    Wt = torch.tensor(Ws, device=dev)
    alpha, c = _params(d)
    at = torch.as_tensor(np.broadcast_to(np.asarray(alpha, np.float64), (len(lens),)).copy()).to(dev)
    ct = torch.as_tensor(np.broadcast_to(np.asarray(c, np.float64), (len(lens),)).copy()).to(dev)
    use_t = d["time"]
    valid = torch.isfinite(flux)
    if use_t:
        valid &= torch.isfinite(time)
    v = torch.nonzero(valid).flatten()                   # packed index of each valid sample
    trend = torch.full((n,), math.nan, device=dev, dtype=torch.float64)
    median = torch.full((n,), math.nan, device=dev, dtype=torch.float64)
    if v.numel():
        start = torch.ones(v.numel(), dtype=torch.bool, device=dev)
        start[1:] = cid[v[1:]] != cid[v[:-1]]
        if use_t:
            start[1:] |= (time[v[1:]] - time[v[:-1]]) > GAP_DAYS
        seg = torch.cumsum(start, 0) - 1
        cnt = torch.bincount(seg)
        first = v[start]
        last = v[torch.cumsum(cnt, 0) - 1]
        live = cnt[seg] >= torch.clamp(Wt[cid[v]] // 3, min=1)
        rank = torch.cumsum(valid, 0) - 1                # compacted position of each sample
        x = flux[v].double()
        tv = time[v] if use_t else None
        for W in sorted(set(Ws)):
            sel = torch.nonzero(live & (Wt[cid[v]] == W)).flatten()
            h = (W - 1) // 2
            for at0 in range(0, sel.numel(), max(1, (1 << 25) // W)):
                i = sel[at0:at0 + max(1, (1 << 25) // W)]  # compacted positions
                p, sg = v[i], seg[i]
                lo = torch.maximum(p - h, first[sg])
                hi = torch.minimum(p + h, last[sg])
                a = rank[lo] + (~valid[lo]).long()       # first valid sample at or after lo
                b = rank[hi]
                j = a[:, None] + torch.arange(W, device=dev)
                inside = j <= b[:, None]
                j = torch.minimum(j, b[:, None])
                if d["window_days"] > 0:
                    inside &= (tv[j] - tv[i][:, None]).abs() <= 0.5 * d["window_days"]
                y = x[j]
                m, mu = _estimate(y, inside, at[cid[p]], ct[cid[p]], d["iters"], d["scale"])
                median[p], trend[p] = m, mu
    return _outputs(trend, median if d["median"] else None,
                    flux.double() / trend if d["detrended"] else None)


def _lower_median(y, inside, k):
    s, _ = torch.sort(torch.where(inside, y, math.inf), dim=1)
    return s.gather(1, k).flatten()


def _estimate(y, inside, alpha, c, iters, scale):
    """Median, scale and asymmetric bisquare iterations of each row's samples."""
    n = inside.sum(1)
    k = ((n - 1) // 2)[:, None]
    m = _lower_median(y, inside, k)
    r = y - m[:, None]
    if scale == "mad":
        s = _lower_median(r.abs(), inside, k)
    else:
        up = inside & (r > 0)
        s = 0.6745 * torch.sqrt((torch.where(up, r, 0.0) ** 2).sum(1) / up.sum(1).clamp(min=1))
    mu = m.clone()
    act = s > 0
    cs = torch.where(act, c * s, 1.0)
    for _ in range(iters):
        r = y - mu[:, None]
        w = r / cs[:, None]
        w = torch.where(w < 0, alpha[:, None] * w, w)
        w = torch.where(inside & (w.abs() < 1), (1 - w * w) ** 2, 0.0)
        sw = w.sum(1)
        act = act & (sw > 0)
        mu = torch.where(act, mu + (w * r).sum(1) / sw.clamp(min=1e-300), mu)
    return m, mu
