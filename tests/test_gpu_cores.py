"""GPU parity of the wide windows' sorted cores (32 aligned windows share a
core summed by its power sums) against the FP64 oracle: medians bit-exact,
trends within the trend tolerance, one result whatever the tile.

The tolerance is the acceptance bound of the main path, relative to
max(|trend|, the window's sample magnitude)."""
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


def _shapes(W, rng):
    """Curves whose groups are regular, cut, sparse, tied, stepped, or badly
    scaled: what decides between the power sums and the direct sums."""
    n = 3 * 64 + W + 700
    noise = rng.normal(0, 1e-3, n)
    t = np.arange(n) * DT
    yield 1 + noise, t                                          # regular
    f = 1 + noise
    f[W // 2 + 70:W // 2 + 70 + 401] = np.nan                   # a gap that splits segments
    yield f, t
    f = 1 + noise
    f[rng.random(n) < 0.3] = np.nan                             # isolated invalid samples
    yield f, t
    yield np.round(1 + noise, 3), t                             # long runs of ties
    yield np.where(np.arange(n) % 900 < 450, 1.0, 0.95) + noise, t   # deep steps
    yield 1 + noise + 3 * (np.arange(n) / n) ** 2, t            # a steep trend
    f = np.full(n, 2.5)
    f[::7] += noise[::7]                                        # mostly constant: no spread
    yield f, t
    f = noise.copy()
    f[::50] = 1e6                                               # far outliers on both sides
    f[25::50] = -1e9
    yield f, t
    yield 1e-15 * (1 + noise), t                                # fifth powers below float32
    yield 1e15 * (1 + noise), t                                 # fifth powers beyond float32
    yield rng.choice(np.array([-0.0, 0.0, 1e-3, -1e-3]), n), t  # signed zeros
    t2 = t.copy()
    t2[n // 2 + 17:] += 0.75                                    # a break in time inside a group
    yield 1 + noise, t2
    yield (1 + noise)[:W + 63], t[:W + 63]                      # barely a core
    yield (1 + noise)[:W // 3 + 1], t[:W // 3 + 1]              # shorter than the window


def core_batch(Ws, seed):
    rng = np.random.default_rng(seed)
    return synth.lightcurves.pack([(np.asarray(f, np.float32), t, W)
                                   for W in Ws for f, t in _shapes(W, rng)])


@pytest.mark.parametrize("Ws,tile", [((137, 143), 1536), ((193, 199, 255), 1536), ((361, 363), 1536), ((721,), 1280),
                                     ((1081, 1441), 512), ((361,), 300)])
def test_cores_against_oracle(torch, umi, oracle_lib, Ws, tile):
    b = core_batch(Ws, 7)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for a, c, it in [(2.0, 5.0, 5), (1.0, 5.0, 5), (10.0, 2.5, 5), (0.5, 5.0, 3), (3.0, 5.0, 1)]:
        g_tr, g_md = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W,
                               launch=umi.LaunchOptions(tile=tile), alpha=a, c=c, iters=it)
        o_tr, o_md = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=a, c=c,
                                              iters=it)
        assert_parity(g_tr, g_md, o_tr, o_md, scale=mag,
                      what="cores W=%s tile %d a=%g c=%g" % (Ws, tile, a, c))


@pytest.mark.parametrize("W", [117, 159, 167, 543, 551])
def test_core_block_counts(torch, umi, oracle_lib, W):
    """Cores whose search tree just fills its levels (16, 64 blocks) or needs
    one more (17, 65); windows that grow and shrink at segment ends, whose edge
    samples differ in number; cut-offs far apart."""
    b = core_batch((W,), 13)
    mag = window_magnitude(b.flux, b.time, b.lengths, b.W, oracle_lib)
    for a, c in [(2.0, 5.0), (16.0, 5.0), (0.25, 5.0)]:
        g_tr, g_md = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, alpha=a, c=c, iters=5)
        o_tr, o_md = oracle_lib.detrend_batch(b.flux, b.time, b.lengths, b.W, alpha=a, c=c, iters=5)
        assert_parity(g_tr, g_md, o_tr, o_md, scale=mag, what="W=%d a=%g" % (W, a))


def test_cores_do_not_depend_on_the_tile(torch, umi):
    b = core_batch((195, 361, 701), 9)
    ref = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=umi.LaunchOptions(tile=1024))
    for lo in [umi.LaunchOptions(tile=257), umi.LaunchOptions(tile=640), umi.LaunchOptions(tile=999),
               umi.LaunchOptions(tile=1301, mode=umi.MODE_PER_CURVE)]:
        out = run_batch(torch, umi, b.flux, b.time, b.lengths, b.W, launch=lo)
        assert np.array_equal(out[0].view(np.uint32), ref[0].view(np.uint32)), lo
        assert np.array_equal(out[1].view(np.uint32), ref[1].view(np.uint32)), lo


@pytest.mark.parametrize("curves,n", [(1, 117), (1, 20000), (8, 20000), (12, 20000), (16, 20000), (40, 20000),
                                      (300, 1200)])
def test_small_batches_take_any_tile(torch, umi, curves, n):
    """Batches that the library cuts into small tiles, one to three a CU, give
    the bits of tiles of 1,024 positions."""
    umi.set_tuning(None)
    rng = np.random.default_rng(curves)
    flux = (1 + 1e-3 * rng.standard_normal(curves * n)).astype(np.float32)
    flux[rng.random(flux.size) < 0.01] = np.nan
    time = np.tile(np.arange(n) * DT, curves)
    auto = run_batch(torch, umi, flux, time, [n] * curves, [361] * curves)
    ref = run_batch(torch, umi, flux, time, [n] * curves, [361] * curves,
                    launch=umi.LaunchOptions(tile=1024))
    for a, r in zip(auto, ref):
        assert np.array_equal(a.view(np.uint32), r.view(np.uint32))


@pytest.mark.parametrize("curves,n", [(36, 18000), (100, 18000), (100, 4408), (300, 4408)])
def test_narrow_windows_take_any_tile(torch, umi, curves, n):
    """Batches of W = 25 of one round of tiles and of several give the bits of
    tiles of 1,536 positions."""
    umi.set_tuning(None)
    rng = np.random.default_rng(n)
    flux = (1 + 1e-3 * rng.standard_normal(curves * n)).astype(np.float32)
    flux[rng.random(flux.size) < 1e-4] = np.nan
    time = np.tile(np.arange(n) * DT, curves)
    auto = run_batch(torch, umi, flux, time, [n] * curves, [25] * curves)
    ref = run_batch(torch, umi, flux, time, [n] * curves, [25] * curves,
                    launch=umi.LaunchOptions(tile=1536))
    for a, r in zip(auto, ref):
        assert np.array_equal(a.view(np.uint32), r.view(np.uint32))


def test_plans_take_the_kernel_their_windows_need(torch, umi):
    """One plan's runs without cores, with cores of middling windows and with
    the widest windows give the direct call's bits."""
    b = core_batch((121, 361, 1441), 11)
    f, t = torch.from_numpy(b.flux).cuda(), torch.from_numpy(b.time).cuda()
    trend, median = torch.empty_like(f), torch.empty_like(f)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan = umi.Plan(f, t, trend, median, max_curves=64, stream=stream)
    off = b.offsets
    try:
        for Ws in [(121,), (121, 361), (121, 361, 1441), (361,), (1441,), (121,)]:
            sel = np.flatnonzero(np.isin(b.W, Ws))
            plan.run(off[sel], b.lengths[sel], b.W[sel])
            stream.synchronize()
            got = (trend.cpu().numpy(), median.cpu().numpy())
            d_tr, d_md = torch.full_like(f, 7.0), torch.full_like(f, 7.0)
            umi.detrend_gather_into(f, t, off[sel], b.lengths[sel], b.W[sel], d_tr, d_md)
            torch.cuda.synchronize()
            for ci in sel:
                sl = slice(off[ci], off[ci] + b.lengths[ci])
                assert np.array_equal(got[0][sl].view(np.uint32), d_tr.cpu().numpy()[sl].view(np.uint32))
                assert np.array_equal(got[1][sl].view(np.uint32), d_md.cpu().numpy()[sl].view(np.uint32))
    finally:
        plan.destroy()
