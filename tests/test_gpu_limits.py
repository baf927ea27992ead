"""Calls at the library's limits on a GPU."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [(1 << 23) - 1, 1 << 23])
def test_as_many_tiles_as_a_launch_has_workgroups_and_one_more(tiles):
    """2^23 workgroups of 512 threads are one more than HIP's 32-bit count of a
    launch's threads holds: that batch goes through the tile queue.  Windows of
    one sample give the sample itself."""
    import torch
    import paper_2604_06602_amd as umi
    g = torch.Generator(device="cuda").manual_seed(tiles)
    flux = torch.randn(tiles, generator=g, device="cuda")
    trend, median = torch.zeros_like(flux), torch.zeros_like(flux)
    umi.detrend_batch_into(flux, None, [tiles], 1, trend, median,
                           launch=umi.LaunchOptions(tile=1))
    torch.cuda.synchronize()
    assert torch.equal(trend, flux) and torch.equal(median, flux)
