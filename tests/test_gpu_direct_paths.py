"""Windows that the sorted cores do not serve, against the FP64 oracle: between
the register networks and the cores (W = 33 to 115), wide ones with asymmetries
outside the cores' range, the very widest, and tiles too small for cores; the
median walk of split tiles at wide windows among them."""
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


@pytest.mark.parametrize("W,alpha,tiles", [(33, 2.0, (1536, 256, 100)), (61, 2.0, (1536, 256, 64)),
                                           (91, 3.0, (1000, 200)), (115, 2.0, (1536, 256, 128, 64)),
                                           (117, 0.2, (1536, 100)), (361, 20.0, (1280, 256, 64)),
                                           (721, 0.2, (512, 128)), (361, 2.0, (63, 32, 1)),
                                           (1441, 2.0, (63, 8)), (1985, 2.0, (0, 63)),
                                           (1987, 2.0, (0,)), (2019, 2.0, (0,)), (2045, 2.0, (0,))])
def test_windows_without_cores(torch, umi, oracle_lib, W, alpha, tiles):
    rng = np.random.default_rng(W)
    some = list(_shapes(W, rng))
    if W > 1500:
        some = some[:5]
    b = synth.lightcurves.pack([(np.asarray(f, np.float32), t, W) for f, t in some])
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    o = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=alpha)
    for tile in tiles:
        g = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, alpha=alpha,
                      launch=umi.LaunchOptions(tile=tile))
        assert_parity(*g, *o, scale=mag, what="W=%d alpha=%g tile=%d" % (W, alpha, tile))


@pytest.mark.parametrize("W,n,tile", [(2017, 1740, 0), (361, 2671, 1)])
def test_tiles_too_small_for_cores_cost_what_direct_sums_do(torch, umi, W, n, tile):
    """Against an asymmetry that never takes cores."""
    rng = np.random.default_rng(5)
    flux = np.where(rng.random(n) < 0.6, 1.0, 1 + 1e-3 * rng.standard_normal(n))
    lo = umi.LaunchOptions(tile=tile)
    direct = call_us(torch, umi, flux, np.arange(n) * DT, 40, W, iters=1, alpha=0.2, launch=lo)
    us = call_us(torch, umi, flux, np.arange(n) * DT, 40, W, iters=1, launch=lo)
    assert us < 1.25 * direct, (us, direct)
