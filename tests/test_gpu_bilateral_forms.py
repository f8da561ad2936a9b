"""Bilateral windows of up to 16 taps: one output a thread on small frames, two on large ones, four there with one or two
taps, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,k,rows", [
    (1, 5, 65, 9, 4), (2, 4, 64, 16, 4), (1, 3, 7, 13, 4), (1, 401, 66, 2, 4),     # cut tiles, windows past every edge
    (401, 1, 3, 3, 16), (401, 17, 5, 8, 16), (401, 16, 4, 4, 16),                   # two outputs a thread: odd and tiny rows
    (401, 16, 4, 1, 16), (401, 17, 5, 2, 16), (401, 1, 3, 2, 16), (402, 3, 70, 1, 16), (3, 800, 195, 2, 16),     # four
    (1, 1030, 1283, 3, 16),
    (401, 9, 6, 9, 4), (1201, 2, 9, 9, 16),                                         # either side of the lines
])
@pytest.mark.parametrize("norm", [-0.01, 0.0004])
def test_against_the_oracle(N, H, W, k, rows, norm):
    rng = np.random.default_rng(N + H + W + k)
    x = rng.uniform(0, 30, (N, H, W)).astype(np.float32)
    gx, gy = (np.exp(-0.5 * ((np.arange(k) - k // 2) / max(k / 3, 0.5)) ** 2).astype(np.float32) for _ in range(2))
    plan = mb.merit_plan_bilateral(N, H, W, k)
    li = plan.launch_info()
    assert li["kernel"] == "merit_bilateral_rows" and li["tile"][1:3] == (rows, 64) and li["block"][0] == (512 if rows == 16 and k > 2 else 256)
    buf = torch.full((N * H * W + 128,), 777.0, device="cuda")
    y = buf[64:64 + N * H * W].view(N, H, W)
    mb.merit_bilateral(plan, torch.from_numpy(x).cuda(), torch.from_numpy(gx).cuda(), torch.from_numpy(gy).cuda(), norm, y)
    assert bool((buf[:64] == 777).all()) and bool((buf[-64:] == 777).all())
    ref = oracle.bilateral(x, gx, gy, norm).astype(np.float64)
    # a weighted mean of values up to 30, weights of a relative error of a few 2^-23 each (an exponent of up to 15 in magnitude)
    assert np.abs(y.cpu().numpy() - ref).max() <= 30 * 2e-6 * 4
