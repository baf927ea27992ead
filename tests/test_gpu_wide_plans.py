"""A plan's step takes what its windows need, whatever the plan could hold."""
from __future__ import annotations

import time as clock

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [361, 601, 721])
def test_a_step_costs_the_same_in_a_plan_for_wider_windows(W):
    import torch
    import paper_2604_06602_amd as umi
    nc, n = 300, 18000
    stream = torch.cuda.Stream()
    flux = 1 + 1e-3 * torch.randn(nc * n, device="cuda")
    time = (torch.arange(n, device="cuda", dtype=torch.float64) * 2 / 1440).repeat(nc)
    trend = torch.empty_like(flux)
    torch.cuda.synchronize()
    us, out = {}, {}
    for max_W in (W, 2047):
        plan = umi.Plan(flux, time, trend, None, max_curves=nc, max_W=max_W, stream=stream)
        try:
            best = np.inf
            for block in range(5):
                stream.synchronize()
                t0 = clock.perf_counter()
                for _ in range(5):
                    plan.run(np.arange(nc) * n, np.full(nc, n), np.full(nc, W))
                stream.synchronize()
                if block:
                    best = min(best, (clock.perf_counter() - t0) / 5)
            us[max_W], out[max_W] = best * 1e6, trend.clone()
            torch.cuda.synchronize()
        finally:
            plan.destroy()
    assert torch.equal(out[W].view(torch.int32), out[2047].view(torch.int32))
    assert us[2047] < 1.3 * us[W], us
