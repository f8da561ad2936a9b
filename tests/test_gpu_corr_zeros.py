"""Correlation beside the image: the zeros left and right of a row, whatever the rows around it and the missing channels of a
last pass hold, on rows that end inside a unit and inside a later chunk's reach, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu

CASES = [
    # N  C   H  W   R  sd
    (1, 20, 5, 70, 4, 8),        # the first chunk reaches past the row's end
    (2, 16, 3, 133, 15, 1),
    (1, 103, 4, 41, 3, 3),       # three residue classes, a last group of seven channels
    (1, 40, 6, 65, 5, 2),        # a last chunk of one pixel
    (2, 260, 5, 47, 3, 1),       # several passes
    (1, 24, 9, 191, 2, 5),
    (1, 40, 6, 72, 5, 2),        # rows of whole units; up to 64 channels, and more
    (2, 64, 5, 40, 4, 1),
    (1, 72, 5, 64, 3, 1),
    (1, 136, 7, 24, 6, 3),
]


@pytest.mark.parametrize("case", CASES)
def test_zeros(case):
    N, C, H, W, R, sd = case
    rng = np.random.default_rng(C + W)
    x1 = (rng.standard_normal((N, C, H, W)) / np.sqrt(C)).astype(np.float16)
    x2 = rng.standard_normal((N, C, H, W)).astype(np.float16)
    plan = mb.merit_plan_correlation(N, C, H, W, R, sd)
    assert plan.launch_info()["kernel"] == "merit_corr_mfma"
    x2[:, :, H // 2] = np.float16(np.inf)                # a row whose neighbours' borders are zeros all the same
    d1, d2 = torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda()
    y = mb.merit_correlation(plan, d1, d2).cpu().numpy().astype(np.float64)
    x2[:, :, H // 2] = 0
    ref = oracle.correlation(x1, x2, R, sd).astype(np.float64)
    # displacements into the row of infinities: not compared; everything else, to one rounding to binary16 and fp32 sums
    p1 = np.arange(H)[:, None] + (np.arange(2 * R + 1)[None] - R) * sd
    keep = np.broadcast_to((p1 != H // 2)[None, :, None, :, None], ref.shape)
    mag = oracle.correlation(np.abs(x1), np.abs(x2), R, sd).astype(np.float64)
    assert np.all((np.abs(y - ref) <= 2.0 ** -10 * np.abs(ref) + (C + 2) * 2.0 ** -23 * mag + 1e-7)[keep])


@pytest.mark.parametrize("R,sd", [(1, 1), (3, 2), (5, 2), (2, 3), (3, 8), (9, 7), (15, 1)])
def test_the_last_columns_of_a_chunk_before_the_last(R, sd):
    """Rows of two and three chunks that end anywhere inside a unit: every column that a product needs is staged, whatever the
    workgroup's LDS held before (infinities, from the call before)."""
    C, H = 24, 6
    rng = np.random.default_rng(R)
    for W in [w for w in range(65, 137) if w % 8] + [191, 193]:
        x1, x2 = (rng.standard_normal((1, C, H, W)).astype(np.float16) for _ in range(2))
        plan = mb.merit_plan_correlation(1, C, H, W, R, sd)
        assert plan.launch_info()["kernel"] == "merit_corr_mfma"
        mb.merit_correlation(plan, *(torch.full((1, C, H, W), float("inf"), device="cuda").half() for _ in range(2)))
        y = mb.merit_correlation(plan, torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda()).cpu().numpy().astype(np.float64)
        ref = oracle.correlation(x1, x2, R, sd).astype(np.float64)
        mag = oracle.correlation(np.abs(x1), np.abs(x2), R, sd).astype(np.float64)
        # one rounding to binary16 and fp32 sums of C products in another order
        assert np.all(np.abs(y - ref) <= 2.0 ** -10 * np.abs(ref) + (C + 2) * 2.0 ** -23 * mag + 1e-7), W
