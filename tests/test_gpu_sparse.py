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
