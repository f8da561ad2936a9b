"""Depthwise layers on the kernel without LDS with one, two and four output rows a thread, and on rows of fewer outputs than
a thread makes, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

# N  C   H   W  k  s  ph pw  rows of a thread
CASES = [
    (3, 40, 31, 21, 3, 1, 1, 1, 1),
    (60, 81, 23, 12, 3, 1, 1, 1, 2),
    (120, 300, 13, 9, 3, 1, 1, 1, 4),
    (30, 300, 15, 11, 5, 1, 2, 2, 2),
    (130, 310, 25, 9, 3, 2, 1, 1, 2),
    (5, 81, 11, 30, 5, 2, 2, 2, 1),
    (200, 3, 24, 1, 3, 1, 1, 1, 1),       # one output a row
    (200, 3, 24, 7, 3, 1, 1, 1, 1),       # seven
    (200, 3, 25, 5, 5, 1, 2, 2, 1),
    (200, 3, 33, 5, 3, 2, 1, 1, 1),       # three
    (1, 400, 2, 3, 5, 2, 4, 4, 1),
    (41, 530, 13, 54, 5, 2, 2, 2, 4),     # four rows at stride 2, the last strip of three
]


@pytest.mark.parametrize("case", CASES)
def test_the_rows_of_a_thread(case):
    _rows_of_a_thread(case)


# large layers at stride 2, to either side of the lines (the plan alone)
@pytest.mark.parametrize("case", [(4, 928, 179, 24, 5, 2, 2, 2, 2), (181, 10, 192, 57, 5, 2, 0, 0, 4), (11, 341, 251, 22, 3, 2, 1, 1, 2),
                                  (60, 5, 317, 762, 3, 2, 1, 1, 4)])
def test_the_rows_of_a_thread_at_stride_2(case):
    _rows_of_a_thread(case)


def _rows_of_a_thread(case):
    N, C, H, W, k, s, ph, pw, rows = case
    li = mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, ph, pw).launch_info()
    assert li["kernel"] == "merit_dwconv_lanes" and li["tile"][2] == rows, li


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case):
    N, C, H, W, k, s, ph, pw, _ = case
    plan = mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, ph, pw)
    rng = np.random.default_rng(H * 100 + W)
    x = rng.standard_normal((N, C, H, W)).astype(np.float16)
    w = (rng.standard_normal((C, k, k)) / k).astype(np.float16)
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    mb.merit_conv2d_depthwise(plan, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = oracle.conv2d_depthwise(x, w, (s, s), (ph, pw)).astype(np.float64)
    mag = oracle.conv2d_depthwise(np.abs(x), np.abs(w), (s, s), (ph, pw)).astype(np.float64)
    # one rounding to binary16 on either side and k*k fp32 sums in another order
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 2.0 ** -10 * np.abs(ref) + k * k * 2.0 ** -23 * mag + 1e-7)
