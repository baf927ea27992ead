"""Curves that are not one long run of samples: many short segments, few valid
samples far apart.  Against the FP64 oracle, and in time against a regular
curve of the same size (generous factors: what they guard against is work that
grows with the number of segments or with the distance between samples)."""
from __future__ import annotations

import time as clock

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import assert_parity, run_batch, window_magnitude

pytestmark = pytest.mark.gpu

DT = 2 / 1440


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.fixture(scope="module")
def umi(torch):
    import paper_2604_06602_amd as _u
    return _u


def call_us(torch, umi, flux, time, n_curves, W, **kw):
    """Best of several timed blocks of calls on one packed batch, in us."""
    f = torch.from_numpy(np.tile(np.asarray(flux, np.float32), n_curves)).cuda()
    t = None if time is None else torch.from_numpy(np.tile(time, n_curves)).cuda()
    out = torch.empty_like(f)
    lens = np.full(n_curves, len(flux))
    best = np.inf
    for block in range(6):
        torch.cuda.synchronize()
        t0 = clock.perf_counter()
        for _ in range(5):
            umi.detrend_batch_into(f, t, lens, W, out, **kw)
        torch.cuda.synchronize()
        if block:
            best = min(best, (clock.perf_counter() - t0) / 5)
    return best * 1e6


def _segmented(W, rng):
    """Curves cut into many segments: of one sample, of lengths around W/3,
    several to a 64-sample word, over invalid samples and over long empty runs."""
    n = 5000
    m = max(1, W // 3)
    steps = np.arange(n) * DT
    yield rng.normal(1, 1e-3, n), np.arange(n) * 1.0              # every sample a segment
    for lo, hi in [(1, 4), (max(1, m - 1), m + 2), (1, 2 * m + 2)]:
        cut = np.zeros(n)
        at = np.cumsum(rng.integers(lo, hi, n))
        cut[at[at < n]] = 0.75
        yield rng.normal(1, 1e-3, n), steps + np.cumsum(cut)
        f = rng.normal(1, 1e-3, n)
        f[rng.random(n) < 0.5] = np.nan
        yield f, steps + np.cumsum(cut)
    f = rng.normal(1, 1e-3, n)                                    # bursts of segments, then nothing
    f[(np.arange(n) // 96) % 3 != 0] = np.nan
    yield f, steps + np.floor(np.arange(n) / 12) * 0.75


@pytest.mark.parametrize("W,tile", [(3, 1536), (7, 1536), (25, 1536), (25, 100), (61, 1000),
                                    (121, 1536), (361, 300), (361, 1536), (1441, 512)])
def test_many_segments_against_oracle(torch, umi, oracle_lib, W, tile):
    rng = np.random.default_rng(17 + W)
    b = synth.lightcurves.pack([(np.asarray(f, np.float32), t, W) for f, t in _segmented(W, rng)])
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=umi.LaunchOptions(tile=tile))
    o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W)
    assert_parity(*g, *o, scale=mag, what="many segments W=%d tile %d" % (W, tile))


@pytest.mark.parametrize("W", [25, 361])
def test_many_segments_cost_no_more_than_one(torch, umi, W):
    n = 18000
    flux = np.random.default_rng(W).normal(1, 1e-3, n)
    one = call_us(torch, umi, flux, np.arange(n) * DT, 40, W)
    many = call_us(torch, umi, flux, np.arange(n) * 1.0, 40, W)
    assert many < 2.5 * one, (many, one)


# steps outwards: four of 256 samples by a wave, then of 16,384 by the
# workgroup, 2,048 a wave, 512 at a time
FAR = [1, 255, 1023, 1025, 1536, 3071, 9000, 17407, 17409, 40000]


def _far_samples(W, tile, rng):
    """A group of valid samples in one tile, W/3 of them only with another far
    outside its staged span: after or before it, on both sides, one sample too
    few, behind a break, with invalid times between."""
    m = max(2, W // 3)
    dt = 1e-6  # no break by itself, however far
    for far in FAR:
        for short in (0, 1):
            for sides in (1, 2, 3):
                n = 2 * (far + tile + W) + max(300, 2 * m + 20)
                here, most = n // 2, m // 2
                f = np.full(n, np.nan)
                f[here:here + most] = rng.normal(1, 1e-3, most)
                rest = m - most - short
                for side, k in ((1, rest if sides == 1 else rest - rest // 2 * (sides == 3)),
                                (2, rest if sides == 2 else rest // 2)):
                    if not sides & side:
                        continue
                    at = here + most + W + tile + far if side == 1 else here - W - tile - far - k
                    f[at:at + k] = rng.normal(1, 1e-3, k)
                t = np.arange(n) * dt
                yield f, t
                if short == 0:
                    u = t.copy()                      # a break where nothing is valid
                    u[here + most + W // 2:] += 0.75
                    yield f, u
                    u = t.copy()                      # invalid by their times
                    g = f.copy()
                    bad = rng.random(n) < 0.3
                    g[bad & np.isnan(f)] = 1.0
                    u[bad & np.isnan(f)] = np.nan
                    yield g, u
    n = 60000                                         # one in 500, breaks among them
    f = np.full(n, np.nan)
    f[::500] = rng.normal(1, 1e-3, f[::500].size)
    t = np.arange(n) * dt
    yield f, t
    for at in (4000, 20001, 20500, 52000):
        t = t.copy()
        t[at:] += 0.75
        yield f, t


@pytest.mark.parametrize("W,tile", [(25, 300), (361, 1536), (361, 64), (2047, 2)])
def test_far_samples_against_oracle(torch, umi, oracle_lib, W, tile):
    rng = np.random.default_rng(23 + W)
    curves = [(np.asarray(f, np.float32), t, W) for f, t in _far_samples(W, tile, rng)]
    if W == 2047:
        curves = curves[:12] + curves[-3:]
    b = synth.lightcurves.pack(curves)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=umi.LaunchOptions(tile=tile))
    o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W)
    live = np.isfinite(o[0])
    assert live.any() and (np.isfinite(b.flux) & ~live).any()
    assert_parity(*g, *o, scale=mag, what="far samples W=%d tile %d" % (W, tile))
    # without times nothing ends a segment
    flux = np.where(np.isfinite(b.time), b.flux, np.nan).astype(np.float32)
    g = run_batch(torch, umi, flux, None, b.lengths, b.W, launch=umi.LaunchOptions(tile=tile))
    o = oracle_lib.detrend_batch(flux, None, b.lengths, b.W)
    assert_parity(*g, *o, scale=mag, what="no times W=%d tile %d" % (W, tile))


@pytest.mark.parametrize("W,every", [(361, 1000), (1441, 1000), (721, 0)])
def test_sparse_curves_cost_little_more_than_full_ones(torch, umi, W, every):
    """One sample in 1,000 valid, or fewer than W/3 among all, without times."""
    rng = np.random.default_rng(W)
    n = 200_000
    flux = rng.normal(1, 1e-3, n)
    keep = rng.random(n) < 1 / every if every else np.isin(np.arange(n), rng.choice(n, W // 3 - 2))
    full = call_us(torch, umi, flux, None, 1, W)
    sparse = call_us(torch, umi, np.where(keep, flux, np.nan), None, 1, W)
    assert sparse < 3 * full, (sparse, full)


def test_segments_of_a_group_do_not_depend_on_the_tile(torch, umi):
    """Groups of wide windows in which one or two segments end: each segment's
    windows have a core of their own, whatever tile the group lies in."""
    rng = np.random.default_rng(41)
    curves = []
    for W in (117, 121, 361, 721):
        n, m = 4000, W // 3
        for lo, hi in [(m, m + 3), (m, 2 * m), (m - 3, m + 4)]:
            at = np.cumsum(rng.integers(lo, hi, n))
            cut = np.zeros(n)
            cut[at[at < n]] = 0.75
            f = rng.normal(1, 1e-3, n)
            f[rng.random(n) < 0.01] = np.nan
            curves.append((f.astype(np.float32), np.arange(n) * DT + np.cumsum(cut), W))
    b = synth.lightcurves.pack(curves)
    ref = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=umi.LaunchOptions(tile=1024))
    assert np.isfinite(ref[0]).any()
    for tile in (1300, 640, 257, 96, 64):
        out = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W,
                        launch=umi.LaunchOptions(tile=tile))
        for a, r in zip(out, ref):
            assert np.array_equal(a.view(np.uint32), r.view(np.uint32)), tile


@pytest.mark.parametrize("W", [361, 1441])
def test_segments_of_half_a_window_cost_little_more_than_one(torch, umi, W):
    n = 18000
    flux = np.random.default_rng(W).normal(1, 1e-3, n)
    one = call_us(torch, umi, flux, np.arange(n) * DT, 100, W)
    cut = np.floor(np.arange(n) / (W // 3 + 20)) * 0.7
    many = call_us(torch, umi, flux, np.arange(n) * DT + cut, 100, W)
    assert many < 1.8 * one, (many, one)


def test_sparse_curves_with_times_cost_little_more_than_full_ones(torch, umi):
    """One sample in 16 valid, no gap over half a day: no break between them."""
    n, W = 18000, 1801
    rng = np.random.default_rng(16)
    flux, t = rng.normal(1, 1e-3, n), np.arange(n) * DT
    full = call_us(torch, umi, flux, t, 100, W)
    sparse = call_us(torch, umi, np.where(rng.random(n) < 1 / 16, flux, np.nan), t, 100, W)
    assert sparse < 1.3 * full, (sparse, full)
