"""Correlation layers whose rows are not whole 8-pixel units, on the MFMA kernel, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


CASES = [
    # N  C   H   W   R  sd
    (1, 16, 40, 9, 2, 1),        # one whole unit and one pixel
    (2, 20, 4, 15, 3, 2),        # one pixel short of two units, channels not a multiple of 8
    (1, 64, 6, 65, 5, 2),        # a second chunk of one pixel
    (1, 130, 3, 71, 3, 3),       # two channel passes, a second chunk of seven pixels
    (1, 32, 5, 41, 15, 1),       # the widest range: displaced past both edges
    (1, 40, 9, 132, 4, 8),       # eight classes, three chunks
    (1, 264, 5, 16, 4, 1),       # one block of pixels, more channels a pass than a wide row leaves room for
    (1, 72, 4, 39, 5, 2),        # two classes of 20 pixels
    (2, 136, 3, 24, 3, 8),       # eight classes of three
    (1, 200, 3, 57, 2, 3),       # one pixel into the last unit of a chunk
    (3, 48, 7, 11, 5, 1),        # rows that start on every 2-byte boundary; the last ends with the tensor
]


@pytest.mark.parametrize("case", CASES)
def test_odd_widths(case):
    N, C, H, W, R, sd = case
    rng = np.random.default_rng(W * 100 + C)
    x1 = (rng.standard_normal((N, C, H, W)) / np.sqrt(C)).astype(np.float16)
    x2 = rng.standard_normal((N, C, H, W)).astype(np.float16)
    plan = mb.merit_plan_correlation(N, C, H, W, R, sd)
    assert plan.launch_info()["kernel"] == "merit_corr_mfma"
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    mb.merit_correlation(plan, torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda(), y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = oracle.correlation(x1, x2, R, sd).astype(np.float64)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.abs(ref) + 1e-3)
    # what lies past a row's end is the next row's: it must not leak in
    x1n, x2n = x1.copy(), x2.copy()
    x1n[:, :, 1:] = np.nan
    x2n[:, :, :, 0] = np.nan
    g = mb.merit_correlation(plan, torch.from_numpy(x1n).cuda(), torch.from_numpy(x2n).cuda()).cpu().numpy()
    cols = np.arange(W)[:, None] + (np.arange(2 * R + 1) - R)[None] * sd
    rows = (np.arange(2 * R + 1) - R) * sd
    for j in range(2 * R + 1):                      # row 0 of the first tensor is clean
        inside = 0 <= rows[j] < H
        want_nan = (cols == 0) & inside
        assert np.array_equal(np.isnan(g[:, 0, :, j, :]), np.broadcast_to(want_nan, g[:, 0, :, j, :].shape))
