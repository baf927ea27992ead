"""Validity, segment breaks and the minimum segment length, decided inside the
estimate kernel from each tile's staged span, against the FP64 oracle: breaks
inside and between 64-sample words and across runs of invalid samples,
segments whose length only samples outside the span decide, dead segments at
the span's borders, with and without times; and the three ways a batch's curve
table reaches the kernel (by value, staged for the tile queue, per curve)."""
from __future__ import annotations

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


def _curves(W, rng):
    n = 4000
    base = lambda: rng.normal(1, 1e-3, n)          # noqa: E731
    t = np.arange(n) * DT
    for at in (1024, 1087, 64 * 31 + 1, 3000):     # one break: word border, word end, inside
        u = t.copy()
        u[at:] += 0.75
        yield base(), u
    u = t.copy()                                   # exactly the threshold: no break
    u[2048:] += 0.5 - DT
    yield base(), u
    f, u = base(), t.copy()                        # breaks after invalid runs of several words
    f[500:700] = np.nan
    f[1500:1530] = np.nan
    u[700:] += 0.3
    u[1530:] += 0.5
    yield f, u
    f = base()                                     # sparse: a window holds few samples
    f[np.arange(n) % 37 != 0] = np.nan
    yield f, t
    f = base()                                     # a few samples, then a long empty run
    f[40:2600] = np.nan
    yield f, t
    f, u = base(), t.copy()                        # short segments, dead and just alive
    m = max(1, W // 3)
    edges = [300, 300 + m - 1, 300 + 2 * m - 1, 1536 - m // 2, 1536 + (m + 1) // 2 - 1, 2500]
    for e in edges:
        u[e:] += 1.0
    yield f, u
    f, u = base(), t.copy()                        # the same among invalid samples and times
    for e in edges:
        u[e:] += 1.0
    f[rng.random(n) < 0.4] = np.nan
    u[rng.random(n) < 0.05] = np.nan
    yield f, u
    f = np.full(n, np.nan)                         # only a handful of samples anywhere
    f[[5, 1700, 1701, 3999]] = [1.0, 1.1, 0.9, 1.2]
    yield f, t


@pytest.mark.parametrize("W,tile", [(25, 1536), (25, 300), (121, 700), (361, 1536), (361, 257),
                                    (361, 64), (721, 1280), (1441, 512), (1441, 128)])
def test_segments_against_oracle(torch, umi, oracle_lib, W, tile):
    rng = np.random.default_rng(3 + W)
    curves = [(np.asarray(f, np.float32), t, W) for f, t in _curves(W, rng)]
    b = synth.lightcurves.pack(curves)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=umi.LaunchOptions(tile=tile))
    o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W)
    assert_parity(*g, *o, scale=mag, what="segments W=%d tile %d" % (W, tile))
    # without times nothing breaks a segment: sparse ones live by their far samples
    flux = np.where(np.isfinite(b.time), b.flux, np.nan).astype(np.float32)
    mag = window_magnitude(flux, None, b.lengths, b.W, oracle_lib)
    g = run_batch(torch, umi, flux, None, b.lengths, b.W, launch=umi.LaunchOptions(tile=tile))
    o = oracle_lib.detrend_batch(flux, None, b.lengths, b.W)
    assert_parity(*g, *o, scale=mag, what="no times W=%d tile %d" % (W, tile))


@pytest.mark.parametrize("n_curves", [1, 2, 32, 33, 40])
def test_table_by_value_and_staged_give_the_same_bits(torch, umi, n_curves):
    """Up to 32 curves the table goes to the kernel by value; an explicit limit
    on the workgroups, per-curve launches or one curve more take the staged
    one.  Empty curves in between, every path of the kernel among the windows."""
    rng = np.random.default_rng(n_curves)
    parts = []
    for i in range(n_curves):
        n = int(rng.integers(200, 3000)) if i % 7 != 3 else 0
        parts.append((rng.normal(1, 1e-3, n).astype(np.float32), np.arange(n) * DT,
                      int([25, 121, 361, 721][i % 4])))
    b = synth.lightcurves.pack(parts)
    for tile in (512, 128):
        ref = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W,
                        launch=umi.LaunchOptions(tile=tile))
        assert np.isfinite(ref[0]).sum() == b.n_samples
        for lo in (umi.LaunchOptions(tile=tile, groups_per_cu=4),
                   umi.LaunchOptions(tile=tile, groups_per_cu=1),
                   umi.LaunchOptions(tile=tile, mode=umi.MODE_PER_CURVE)):
            out = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=lo)
            assert np.array_equal(out[0].view(np.uint32), ref[0].view(np.uint32)), (tile, lo)
            assert np.array_equal(out[1].view(np.uint32), ref[1].view(np.uint32)), (tile, lo)
