"""Sorted cores on values that leave the ordinary way, against the FP64 oracle
and, in time, against ordinary noise: medians of zero of either sign among ties,
and cores most of whose samples are equal."""
from __future__ import annotations

import numpy as np
import pytest

import synth
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


def _zeros(n, rng):
    """Values whose windows' medians are zero."""
    yield np.round(1e-3 * rng.standard_normal(n), 3)
    yield rng.choice(np.array([-0.0, 0.0, 1e-3, -1e-3]), n)
    yield np.where(rng.random(n) < 0.5, -0.0, 1e-3 * np.abs(rng.standard_normal(n)))
    yield np.where(rng.random(n) < 0.5, 0.0, -1e-3 * np.abs(rng.standard_normal(n)))
    yield np.full(n, -0.0)


@pytest.mark.parametrize("W", [117, 361, 1441])
def test_medians_of_zero(torch, umi, oracle_lib, W):
    rng = np.random.default_rng(W)
    n = 2 * W + 700
    b = synth.lightcurves.pack([(f.astype(np.float32), np.arange(n) * DT, W)
                                for f in _zeros(n, rng)])
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W)
    o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W)
    assert_parity(*g, *o, scale=mag, what="zero medians W=%d" % W)


def test_medians_of_zero_cost_little_more_than_others(torch, umi):
    n, W = 18000, 361
    rng = np.random.default_rng(2)
    noise = 1e-3 * rng.standard_normal(n)
    other = call_us(torch, umi, 1 + noise, np.arange(n) * DT, 100, W)
    zero = call_us(torch, umi, np.round(noise, 3), np.arange(n) * DT, 100, W)
    assert zero < 2.2 * other, (zero, other)


@pytest.mark.parametrize("W", [117, 361, 1441])
def test_mostly_equal_cores(torch, umi, oracle_lib, W):
    """Half to all but a few of a core's samples equal, the rest noise on both
    sides, on one side, or far out."""
    rng = np.random.default_rng(31 + W)
    n = 2 * W + 700
    curves = []
    for share in (0.6, 0.75, 0.9, 0.97, 0.999):
        for rest in (1e-3 * rng.standard_normal(n), 1e-3 * np.abs(rng.standard_normal(n)),
                     -1e-3 * np.abs(rng.standard_normal(n)), 1e-3 * rng.standard_cauchy(n)):
            curves.append((np.where(rng.random(n) < share, 1.0, 1 + rest).astype(np.float32),
                           np.arange(n) * DT, W))
    b = synth.lightcurves.pack(curves)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for a, c in [(2.0, 5.0), (10.0, 2.5), (1.0, 5.0)]:
        g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, alpha=a, c=c)
        o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=a, c=c)
        assert_parity(*g, *o, scale=mag, what="mostly equal W=%d a=%g" % (W, a))


@pytest.mark.parametrize("share", [0.75, 0.97])
def test_mostly_equal_cores_cost_little_more_than_others(torch, umi, share):
    n, W = 18000, 1441
    rng = np.random.default_rng(4)
    noise = 1 + 1e-3 * rng.standard_normal(n)
    other = call_us(torch, umi, noise, np.arange(n) * DT, 40, W)
    equal = call_us(torch, umi, np.where(rng.random(n) < share, 1.0, noise), np.arange(n) * DT,
                    40, W)
    assert equal < 3 * other, (equal, other)
