"""Separable filter on rows that are not whole 16-byte groups, against the oracle; the border is replicated from the
row's true last pixel whatever the last group holds.  Tolerance: 2k fp32 multiply-adds of at most |kx| |ky| max|x|."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [3, 4, 5, 6, 7, 63, 65, 66, 67, 127, 190])
@pytest.mark.parametrize("k", [1, 3, 8, 17, 32])
def test_widths(W, k):
    N, H = 2, 21
    rng = np.random.default_rng(100 * W + k)
    x = rng.uniform(0, 255, (N, H, W)).astype(np.float32)
    kx, ky = (rng.standard_normal(k).astype(np.float32) for _ in range(2))
    plan = mb.merit_plan_sepfilter(N, H, W, k)
    buf = torch.full((N * H * W + 128,), 777.0, device="cuda")
    y = buf[64:64 + N * H * W].view(N, H, W)
    mb.merit_sepfilter(plan, torch.from_numpy(x).cuda(), torch.from_numpy(kx).cuda(), torch.from_numpy(ky).cuda(), y)
    assert bool((buf[:64] == 777).all()) and bool((buf[-64:] == 777).all())
    ref = oracle.sepfilter(x, kx, ky).astype(np.float64)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 1e-5 * np.abs(kx).sum() * np.abs(ky).sum() * x.max())
