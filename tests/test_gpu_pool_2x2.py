"""2x2 / stride 2 pooling on rows that are not whole 16-byte vectors, a row a group and four, against the oracle: the maxima to
the bit, the means but for the order of their three additions."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

CASES = [
    # N  C    H   W    rows of a group (0: the tile kernel)
    (2, 106, 11, 13, 0),
    (5, 300, 9, 9, 0),             # 24000 outputs
    (30, 300, 9, 9, 1),            # a last input row and column that no window has
    (3, 606, 38, 13, 1),
    (2, 34, 57, 85, 1),
    (1, 71, 32, 301, 1),           # two chunks of 128 columns
    (8, 512, 28, 28, 1),
    (1, 4096, 29, 29, 1),
    (8, 500, 28, 28, 1),
    (8, 1, 65536, 10, 4),          # a row a group is too long a list
]


# large launches, to either side of the line (the plan alone)
LARGE = [(38, 157, 94, 262, 4), (204, 15, 705, 34, 4), (51, 194, 60, 754, 1), (203, 284, 228, 10, 1), (100, 15, 705, 34, 1)]


@pytest.mark.parametrize("case", CASES + LARGE)
def test_rows_of_a_group(case):
    N, C, H, W, rows = case
    li = mb.merit_plan_pool2d(N, C, H, W, 2, 2, 2, 2, 0, 0, 1).launch_info()
    if rows == 0:
        assert li["kernel"] == "merit_pool2d_tile<avg>"
    else:
        assert li["kernel"] == "merit_pool2d_lanes2_s2<avg,2>" and li["tile"][2] == rows, li


@pytest.mark.gpu
@pytest.mark.parametrize("avg", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case, avg):
    N, C, H, W, _ = case
    x = np.random.default_rng(H * W).standard_normal((N, C, H, W)).astype(np.float32)
    plan = mb.merit_plan_pool2d(N, C, H, W, 2, 2, 2, 2, 0, 0, avg)
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    mb.merit_pool2d(plan, torch.from_numpy(x).cuda(), y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = oracle.pool2d(x, (2, 2), (2, 2), (0, 0), "avg" if avg else "max")
    if avg:       # sums of four in another order: three roundings of at most 2^-24 of the magnitudes' sum
        mag = oracle.pool2d(np.abs(x), (2, 2), (2, 2), (0, 0), "avg")
        assert np.all(np.abs(y.cpu().numpy() - ref) <= 2.0 ** -22 * mag)
    else:
        assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(30, 300, 9, 9), (2, 34, 57, 85), (2, 4, 131072, 10)])
def test_nan_and_infinities_stay_in_their_windows(case):
    """A maximum passes over NaN unless it is all there is, a mean with one is one; the windows beside are as without."""
    N, C, H, W = case
    x = np.random.default_rng(7).standard_normal((N, C, H, W)).astype(np.float32)
    x[::2, 1, 0, 3], x[:, 2, 2:4, 2:4], x[:, 3, 4, 5], x[0, :, 6, 7], x[1, :, 6, 6] = np.nan, np.nan, np.inf, -np.inf, np.finfo(np.float32).min
    win = x[:, :, :H // 2 * 2, :W // 2 * 2].reshape(N, C, H // 2, 2, W // 2, 2)
    dx = torch.from_numpy(x).cuda()
    top = mb.merit_pool2d(mb.merit_plan_pool2d(N, C, H, W, 2, 2, 2, 2, 0, 0, 0), dx).cpu().numpy()
    want = np.fmax(np.fmax(win[:, :, :, 0, :, 0], win[:, :, :, 0, :, 1]), np.fmax(win[:, :, :, 1, :, 0], win[:, :, :, 1, :, 1]))
    assert np.array_equal(top, want, equal_nan=True) and np.isnan(top[:, 2, 1, 1]).all()
    mean = mb.merit_pool2d(mb.merit_plan_pool2d(N, C, H, W, 2, 2, 2, 2, 0, 0, 1), dx).cpu().numpy()
    want = win.astype(np.float64).mean(axis=(3, 5)).astype(np.float32)
    finite = np.isfinite(want)
    assert np.array_equal(mean[~finite], want[~finite], equal_nan=True)
    mag = np.abs(win).astype(np.float64).mean(axis=(3, 5))[finite]
    assert np.all(np.abs(mean[finite] - want[finite]) <= 2.0 ** -22 * mag)   # three roundings of at most 2^-24 of the magnitudes' sum
