"""Time windows (window_days) at every cadence against the FP64 oracle: even,
random, in blocks of different density, in bursts, with repeated times and with
anything in the times of invalid samples; and in time against even cadence
(generous factors: what they guard against is work that grows with the distance
between a window's ends and the index window's, or with how much the windows of
neighbouring samples differ)."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from tests.test_gpu_cores import _shapes
from tests.test_gpu_parity import assert_parity, run_batch, window_magnitude
from tests.test_gpu_sparse import call_us

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


def cadences(n, rng):
    i = np.arange(n)
    yield i * DT
    yield np.sort(rng.random(n)) * n * DT                                # random
    yield np.cumsum(np.where((i // 700) % 2 == 0, DT, DT / 6))           # blocks of two densities
    yield np.cumsum(np.where((i // 90) % 2 == 0, DT, DT * 15))
    yield np.cumsum(np.where(i % 60 == 0, DT * 30, DT / 4))              # bursts
    yield np.floor(i / 7) * 7 * DT                                       # repeated times
    yield i * DT + 0.75 * (i >= n // 2 + 17)                             # a break


def batch_of(W, rng, dirty):
    n = 3 * 64 + W + 900
    curves = []
    for t in cadences(n, rng):
        f = 1 + 1e-3 * rng.standard_normal(n)
        if dirty:
            bad = rng.random(n) < 0.3
            f[bad] = np.nan
            f[n // 3:n // 3 + 130] = np.nan                              # words without a sample
            t = t.copy()
            t[np.isnan(f)] = rng.choice([0.0, -1e9, 1e9, np.nan, np.inf, t[n // 2]],
                                        int(np.isnan(f).sum()))
        curves.append((f.astype(np.float32), t, W))
    return synth.lightcurves.pack(curves)


@pytest.mark.parametrize("scale", ["upper_rms", "mad"])
@pytest.mark.parametrize("W,tile", [(25, 1536), (121, 1536), (121, 100), (361, 1280), (1081, 768)])
@pytest.mark.parametrize("dirty", [False, True])
def test_time_windows_at_any_cadence(torch, umi, oracle_lib, W, tile, scale, dirty):
    b = batch_of(W, np.random.default_rng(5 + W), dirty)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for share in (1e-9, 0.05, 0.4, 0.9, 3.0):  # of the even cadence's index window
        L = share * W * DT
        g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, window_days=L, scale=scale,
                      launch=umi.LaunchOptions(tile=tile))
        o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, window_days=L, scale=scale)
        assert_parity(*g, *o, scale=mag, what="W=%d tile %d L=%g %s" % (W, tile, L, scale))


def test_short_time_windows_cost_little_more_than_index_windows(torch, umi):
    n, W = 18000, 1081
    rng = np.random.default_rng(1)
    flux, time = 1 + 1e-3 * rng.standard_normal(n), np.arange(n) * DT
    index = call_us(torch, umi, flux, time, 40, W)
    short = call_us(torch, umi, flux, time, 40, W, window_days=0.05)
    assert short < 4 * index, (short, index)


@pytest.mark.parametrize("W", [121, 361, 1081])
def test_uneven_windows_of_any_values(torch, umi, oracle_lib, W):
    """Windows of neighbouring samples that differ by more samples than a group
    of windows has slots for, over ties, steps, outliers and signed zeros."""
    rng = np.random.default_rng(29 + W)
    curves = []
    for f, t in _shapes(W, rng):
        n = len(f)
        u = np.sort(rng.random(n)) * (t[-1] - t[0])
        burst = np.cumsum(np.where(np.arange(n) % 60 == 0, DT * 30, DT / 4))
        curves += [(np.asarray(f, np.float32), x, W) for x in (u, burst)]
    b = synth.lightcurves.pack(curves)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for a, c, share in [(2.0, 5.0, 0.6), (1.0, 5.0, 0.3), (10.0, 2.5, 0.6)]:
        L = share * W * DT
        g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, alpha=a, c=c, window_days=L)
        o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=a, c=c, window_days=L)
        assert_parity(*g, *o, scale=mag, what="uneven W=%d a=%g L=%g" % (W, a, L))


@pytest.mark.parametrize("W,kind", [(1081, "random"), (361, "bursts")])
def test_uneven_windows_cost_little_more_than_even_ones(torch, umi, W, kind):
    n, L = 18000, 0.9 * W / 1081
    rng = np.random.default_rng(3)
    flux = 1 + 1e-3 * rng.standard_normal(n)
    uneven = (np.sort(rng.random(n)) * n * DT if kind == "random" else
              np.cumsum(np.where(np.arange(n) % 60 == 0, DT * 30, DT / 4)))
    even = call_us(torch, umi, flux, np.arange(n) * DT, 40, W, window_days=L)
    us = call_us(torch, umi, flux, uneven, 40, W, window_days=L)
    assert us < 4 * even, (us, even)


@pytest.mark.parametrize("W,n_curves,n", [(121, 40, 18000), (361, 40, 18000), (121, 1, 1229)])
def test_windows_of_72_and_73_samples_cost_what_82_do(torch, umi, W, n_curves, n):
    """At 0.1 days the windows' ends fall on samples, whose times are rounded:
    neighbouring windows differ by a sample, and the group's core by two."""
    rng = np.random.default_rng(7)
    flux, t = 1 + 1e-3 * rng.standard_normal(n), np.arange(n) * DT
    other = call_us(torch, umi, flux, t, n_curves, W, window_days=0.115)
    us = call_us(torch, umi, flux, t, n_curves, W, window_days=0.1)
    assert us < 1.6 * other, (us, other)


@pytest.mark.parametrize("days", [0.055, 0.0612, 0.08, 0.1, 0.12])
def test_short_cores_of_time_windows(torch, umi, oracle_lib, days):
    """Cores of 9 to 60 samples, with up to as many samples beside them."""
    rng = np.random.default_rng(11)
    curves = []
    for W in (121, 361):
        for f, t in _shapes(W, rng):
            n = len(f)
            for u in (t, t + 0.3 * DT * rng.random(n), np.cumsum(rng.uniform(0.5, 1.5, n)) * DT):
                curves.append((np.asarray(f, np.float32), np.sort(u), W))
    b = synth.lightcurves.pack(curves)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for a, c in [(2.0, 5.0), (1.0, 2.0)]:
        g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, alpha=a, c=c, window_days=days)
        o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=a, c=c, window_days=days)
        assert_parity(*g, *o, scale=mag, what="short cores %g days a=%g" % (days, a))
