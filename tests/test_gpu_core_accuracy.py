"""Accuracy of wide windows (sorted cores) where the values within the cut-offs
are a small part of the spread: steps, eclipses, flares, mixtures and saw teeth of
3 to 300 times the noise, against the FP64 oracle.

Tolerances: the acceptance bound of the main path for every sample, and for a
curve's rms error 5e-7, eight times float32's 2^-24 at values of about 1, which
window sums of float32 residuals keep to whatever the spread is.  At alpha of 10
and more the iterations do not contract on such curves and multiply any
rounding: windows summed sample by sample are off by up to 4e-5 there too."""
from __future__ import annotations

import numpy as np
import pytest

from tests.test_gpu_parity import REL_TOL, run_batch

pytestmark = pytest.mark.gpu


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


def shapes(n, rng, s=1e-3):
    x, i = 1 + s * rng.standard_normal(n), np.arange(n)
    for a in (3, 30, 300):
        a *= s
        yield x - a * ((i % 900) >= 450)
        yield x - a * ((i % 97) >= 48)
        yield x + a * rng.integers(0, 2, n // 40 + 1)[i // 40]
        yield x + a * rng.integers(-1, 2, n // 40 + 1)[i // 40]
        yield x - a * (np.abs((i % 400) - 200) < 40)
        yield x + a * ((i % 300) / 300)
        yield x + a * np.exp(-(i % 500) / 20.0)
        yield x + a * (rng.random(n) < 0.3)
        yield x + a * (rng.random(n) < 0.45)
        yield x - a * (rng.random(n) < 0.45)


@pytest.mark.parametrize("W", [117, 121, 241, 361, 721, 1441])
@pytest.mark.parametrize("alpha,c", [(2.0, 5.0), (1.0, 5.0), (0.25, 5.0), (3.0, 1.0)])
def test_spread_far_beyond_the_cut_offs(torch, umi, oracle_lib, W, alpha, c):
    n = 2 * W + 1000
    f = np.array(list(shapes(n, np.random.default_rng(W))), np.float32)
    lens, Ws = [n] * len(f), [W] * len(f)
    tr, _ = run_batch(torch, umi, f.ravel(), None, lens, Ws, alpha=alpha, c=c)
    o, _ = oracle_lib.detrend_batch(f.ravel(), None, lens, Ws, alpha=alpha, c=c)
    err = np.abs(tr - o).reshape(f.shape)
    assert err.max() <= REL_TOL, (np.unravel_index(err.argmax(), err.shape), err.max())
    rms = np.sqrt((err ** 2).mean(1))
    assert rms.max() <= 5e-7, (rms.argmax(), rms.max())
