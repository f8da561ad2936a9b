"""Depthwise layers on the kernel without LDS, against the oracle: rows that are not whole units, strips cut by the
image's end, paddings beyond the window, the tensor's first and last units."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


# (as many planes as send layers of these sizes to this kernel)
CASES = [
    # N  C   H   W  k  s  ph pw
    (120, 81, 5, 9, 3, 1, 1, 1),        # a unit and one output
    (120, 81, 9, 15, 3, 1, 0, 0),
    (120, 81, 7, 8, 3, 1, 0, 1),
    (120, 81, 12, 23, 3, 2, 1, 1),
    (120, 81, 3, 8, 3, 2, 1, 1),        # one unit a row, two rows
    (120, 81, 13, 17, 5, 1, 2, 2),
    (120, 81, 10, 24, 5, 1, 4, 4),      # outputs that see only padding in part of the window
    (120, 81, 11, 30, 5, 2, 2, 2),
    (120, 81, 6, 8, 5, 2, 0, 4),
    (120, 81, 4, 8, 3, 1, 2, 6),        # whole units of padding
    (4, 40, 20, 65, 3, 1, 1, 1),
]


@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case):
    N, C, H, W, k, s, ph, pw = case
    plan = mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, ph, pw)
    assert plan.launch_info()["kernel"] == "merit_dwconv_lanes", plan.launch_info()
    rng = np.random.default_rng(H * 100 + W)
    x = rng.standard_normal((N, C, H, W)).astype(np.float16)
    w = (rng.standard_normal((C, k, k)) / k).astype(np.float16)
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    mb.merit_conv2d_depthwise(plan, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = oracle.conv2d_depthwise(x, w, (s, s), (ph, pw)).astype(np.float64)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.abs(ref) + 1e-3)
    # rows and planes next to each other: a NaN reaches exactly the windows that hold it
    x[0, 0, H - 1, W - 1] = x[N - 1, C - 1, H - 1, W - 1] = np.nan
    got = np.isnan(mb.merit_conv2d_depthwise(plan, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()).cpu().numpy())
    oy, ox = np.meshgrid(np.arange(got.shape[2]), np.arange(got.shape[3]), indexing="ij")
    want = np.zeros_like(got)
    want[0, 0] = want[N - 1, C - 1] = ((oy * s - ph <= H - 1) & (oy * s - ph + k > H - 1) & (ox * s - pw <= W - 1) & (ox * s - pw + k > W - 1))
    assert np.array_equal(got, want)
