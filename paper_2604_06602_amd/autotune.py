"""Autotuner for the persistent launch: tile size (and with it the per-window
work split) and workgroups per CU, per W bucket and batch-size bucket.

For each window-size bucket the tuner times every candidate (tile, groups per
CU) on a large synthetic batch of that W with HIP events on the launch stream
and keeps the fastest; then, for batches of one, four and sixteen
20,000-sample curves, it times tiles from the largest down to 64 positions
(tiles of at most 256 positions split each window without a sorted core over 2, 4
or 8 lanes) and
keeps the fastest call for each batch size.  The winners are written as a
tuning table -- the text format of ``umi_set_tuning`` ("W_max tile
groups_per_cu [samples_max]" per line) -- to a JSON cache keyed by GPU
architecture and library version.  ``apply()`` loads the cached table for the
current device into the library.

Usage on a GPU:  python -m paper_2604_06602_amd.autotune [--out PATH]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

from . import _lib

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT_CACHE = os.path.join(HERE, "tuning", "umi_tuning.json")
STAGE_MAX = 2048          # largest staged span (tile + W - 1) of the main kernel
THREADS = 512             # threads per main-kernel workgroup
BUCKETS = [(31, 25), (127, 121), (383, 361), (767, 721), (2047, 1441)]  # (W_max, W tried)
GROUPS = [1, 2, 3, 4]
SPLIT_TILES = [256, 128, 64]   # tiles that split a window without a core over 2, 4 and 8 lanes
# small batches (curves of SMALL_LENGTH samples): (curves, samples_max of the
# tuning row it decides); larger batches take the bucket's general row
SMALL_LENGTH = 20000
SMALL_BATCHES = [(1, 40000), (4, 160000), (16, 640000)]


MAX_TILE = 3 * THREADS    # at most three output positions per lane


def max_tile(W: int) -> int:
    return max(1, min(MAX_TILE, STAGE_MAX - (W - 1)))


TIE = 0.015


def default_tile(W: int) -> int:
    """The library's built-in tile: the largest one, cut back to whole passes
    of the workgroup when the last pass would leave most lanes idle."""
    fill = max_tile(W)
    rem = fill % THREADS
    return fill - rem if fill >= THREADS and rem < THREADS // 2 else fill


def tile_candidates(W: int):
    mt = max_tile(W)
    c = {t for t in range(THREADS // 2, mt + 1, THREADS // 2)}
    c.add(mt)
    c.add(default_tile(W))
    return sorted(c)


def small_batch_candidates(W: int):
    """Tiles for a batch too small to fill the GPU: the large-batch ones of at
    least 512 positions, the split tiles, and what the library's own rule takes
    between them."""
    c = {t for t in tile_candidates(W) if t >= THREADS}
    c.update(t for t in SPLIT_TILES + [320, 384, 640] if t <= max_tile(W))
    c.add(max_tile(W))
    return sorted(c)


def _arch():
    import torch
    p = torch.cuda.get_device_properties(torch.cuda.current_device())
    return getattr(p, "gcnArchName", "unknown").split(":")[0]


def _workload(W: int, n_curves: int, length: int, seed: int = 0):
    """A synthetic batch on the device: level 1 with 1e-3 noise and a slow
    sinusoid, 2-min cadence, no gaps (timing depends on W and lengths)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = n_curves * length
    t = torch.arange(length, device="cuda", dtype=torch.float64) * (2.0 / 1440.0)
    flux = 1.0 + 1e-3 * torch.randn(n, device="cuda", generator=g, dtype=torch.float32)
    flux += (1e-3 * torch.sin(2 * torch.pi * t / 2.7)).float().repeat(n_curves)
    time_ = t.repeat(n_curves).contiguous()
    lengths = [length] * n_curves
    return flux.contiguous(), time_, lengths, [W] * n_curves


def time_candidate(flux, time_, lengths, Ws, trend, tile, gpc, steps=5, warmup=2):
    import torch
    opt = _lib.LaunchOptions(mode=_lib.MODE_PERSISTENT, tile=tile, groups_per_cu=gpc)
    stream = torch.cuda.current_stream()
    for _ in range(warmup):
        _lib.detrend_batch_into(flux, time_, lengths, Ws, trend, None, launch=opt, stream=stream)
    a = torch.cuda.Event(enable_timing=True)
    b = torch.cuda.Event(enable_timing=True)
    a.record(stream)
    for _ in range(steps):
        _lib.detrend_batch_into(flux, time_, lengths, Ws, trend, None, launch=opt, stream=stream)
    b.record(stream)
    torch.cuda.synchronize()
    return a.elapsed_time(b) / steps


def tune(n_curves=400, length=20000, steps=5, log=print):
    import torch
    rows, detail = [], {}
    _lib.set_tuning(None)
    for w_max, W in BUCKETS:
        # small batches first: their rows precede the bucket's general row
        for curves, samples_max in SMALL_BATCHES:
            flux, time_, lengths, Ws = _workload(W, curves, SMALL_LENGTH, seed=curves)
            trend = torch.empty_like(flux)
            # the library's workgroups per CU, so that the call takes the path
            # (by value, without a queue) that it takes in use
            results = sorted((time_candidate(flux, time_, lengths, Ws, trend, tile, 0,
                                             steps=max(steps, 20)), tile)
                             for tile in small_batch_candidates(W))
            # a row serves batches of up to twice the size timed here: of equally
            # fast tiles the largest, which that batch still runs at once
            tile = max(t for m, t in results if m <= results[0][0] * (1 + 2 * TIE))
            rows.append((w_max, tile, GROUPS[-1], samples_max))
            detail["%d/%d" % (w_max, samples_max)] = {
                "W": W, "curves": curves, "length": SMALL_LENGTH, "best_ms": results[0][0],
                "candidates": [{"tile": t, "groups_per_cu": GROUPS[-1], "ms": m}
                               for m, t in results]}
            log("W<=%d (W=%d), %d curve(s) of %d: tile %d, %.3f ms per call (tile %d: %.3f ms)"
                % (w_max, W, curves, SMALL_LENGTH, tile, results[0][0],
                   results[-1][1], results[-1][0]))
            del flux, time_, trend
        flux, time_, lengths, Ws = _workload(W, n_curves, length)
        trend = torch.empty_like(flux)
        results = []
        for tile in tile_candidates(W):
            for gpc in GROUPS:
                ms = time_candidate(flux, time_, lengths, Ws, trend, tile, gpc, steps)
                results.append((ms, tile, gpc))
        results.sort()
        best = results[0]
        # timing noise is a few percent: keep the built-in default unless a
        # candidate beats it by more than TIE
        default = [r for r in results if r[1] == default_tile(W) and r[2] == GROUPS[-1]]
        if default and default[0][0] <= best[0] * (1 + TIE):
            best = default[0]
        rows.append((w_max, best[1], best[2], 0))
        detail[str(w_max)] = {"W": W, "best_ms": best[0],
                              "candidates": [{"tile": t, "groups_per_cu": g, "ms": m}
                                             for m, t, g in results]}
        log("W<=%d (W=%d): tile %d, %d groups/CU, %.3f ms (worst %.3f ms)"
            % (w_max, W, best[1], best[2], best[0], results[-1][0]))
        del flux, time_, trend
        torch.cuda.empty_cache()
    table = "".join("%d %d %d %d\n" % r if r[3] else "%d %d %d\n" % r[:3] for r in rows)
    return table, detail


def cache_key() -> str:
    return "%s/%s" % (_arch(), _lib.version())


def save(table: str, detail: dict, path: str = DEFAULT_CACHE):
    data = {}
    if os.path.exists(path):
        with open(path) as fh:
            data = json.load(fh)
    data[cache_key()] = {"table": table, "detail": detail,
                         "tuned_at": time.strftime("%Y-%m-%dT%H:%M:%S")}
    os.makedirs(os.path.dirname(path), exist_ok=True)
    with open(path, "w") as fh:
        json.dump(data, fh, indent=1, sort_keys=True)


def load_table(path: str = DEFAULT_CACHE):
    """The cached table for this device and library version, or None."""
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        data = json.load(fh)
    entry = data.get(cache_key())
    return None if entry is None else entry["table"]


def apply(path: str = DEFAULT_CACHE) -> bool:
    """Load the cached table into the library; False if there is none."""
    table = load_table(path)
    if table is None:
        return False
    _lib.set_tuning(table)
    return True


def main(argv=None):
    ap = argparse.ArgumentParser(description="tune tile size and workgroups per CU per W bucket")
    ap.add_argument("--out", default=DEFAULT_CACHE)
    ap.add_argument("--curves", type=int, default=400)
    ap.add_argument("--length", type=int, default=20000)
    ap.add_argument("--steps", type=int, default=5)
    args = ap.parse_args(argv)
    table, detail = tune(args.curves, args.length, args.steps,
                         log=lambda m: print(m, flush=True))
    save(table, detail, args.out)
    print(table, end="")
    return 0


if __name__ == "__main__":
    sys.exit(main())
