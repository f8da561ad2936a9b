"""Tile requests of the separable filter: the staged rows asked for, on every form, and the result of the plan without one."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

# N, H, W, k, staged rows asked for
CASES = [(1, 200, 232, 20, 96), (4, 1080, 1920, 20, 96), (4, 1080, 1920, 28, 65), (1, 200, 233, 17, 90), (2, 130, 70, 30, 96),
         (2, 130, 70, 32, 67), (4, 1080, 1920, 20, 64), (1, 200, 232, 20, 40), (4, 1080, 1920, 9, 64), (1, 90, 100, 16, 19)]


@pytest.mark.parametrize("case", CASES)
def test_the_rows_asked_for(case):
    N, H, W, k, rows = case
    li = mb.merit_plan_sepfilter(N, H, W, k).set_tile((0, rows)).launch_info()
    assert li["tile"][1] == (rows - k + 1) // 4 * 4, li


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case):
    N, H, W, k, rows = case
    rng = np.random.default_rng(rows)
    x = rng.uniform(0, 255, (N, H, W)).astype(np.float32)
    kx, ky = (rng.standard_normal(k).astype(np.float32) for _ in range(2))
    plan = mb.merit_plan_sepfilter(N, H, W, k).set_tile((0, rows))
    y = mb.merit_sepfilter(plan, *(torch.from_numpy(a).cuda() for a in (x, kx, ky))).cpu().numpy()
    # 2k fp32 multiply-adds of at most |kx| |ky| max|x|
    ref = oracle.sepfilter(x, kx, ky).astype(np.float64)
    assert np.all(np.abs(y - ref) <= 1e-5 * np.abs(kx).sum() * np.abs(ky).sum() * x.max())
