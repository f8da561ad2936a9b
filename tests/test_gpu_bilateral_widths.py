"""Bilateral filter on rows that are not whole 16-byte groups, against the oracle (tolerance of the parity tests: weight
error plus the fp32 sums, over each window's own range)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [3, 4, 5, 6, 7, 63, 65, 66, 67, 131])
@pytest.mark.parametrize("k", [1, 4, 9, 16, 21])
def test_widths(W, k):
    H = 19
    rng = np.random.default_rng(100 * W + k)
    x = (rng.integers(0, 3, (1, H, W)) * 80 + rng.normal(0, 6, (1, H, W))).astype(np.float32)
    g = np.exp(-0.5 * ((np.arange(k) - k // 2) / 2.0) ** 2).astype(np.float32)
    plan = mb.merit_plan_bilateral(1, H, W, k)
    buf = torch.full((H * W + 128,), 777.0, device="cuda")
    y = buf[64:64 + H * W].view(1, H, W)
    dg = torch.from_numpy(g).cuda()
    mb.merit_bilateral(plan, torch.from_numpy(x).cuda(), dg, dg, -1 / 800, y)
    assert bool((buf[:64] == 777).all()) and bool((buf[-64:] == 777).all())
    ref = oracle.bilateral(x, g, g, -1 / 800).astype(np.float64)
    c = k // 2
    pad = np.pad(x[0], ((c, k - 1 - c), (c, k - 1 - c)), mode="edge")
    win = np.lib.stride_tricks.sliding_window_view(pad, (k, k))
    span, top = win.max((2, 3)) - win.min((2, 3)), np.abs(win).max((2, 3))
    assert np.all(np.abs(y.cpu().numpy()[0] - ref[0]) <= (2e-5 + 1.2e-7 * k * k) * span + 2.4e-7 * top)
