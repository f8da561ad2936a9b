"""16x16 blocks with a search range of 8 on the two-blocks-per-wavefront row scan: bit-exact, ragged frames included."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(16, 16), (50, 100), (41, 96), (64, 260), (9, 20), (130, 132)])
@pytest.mark.parametrize("kind", ["noise", "moved", "flat"])
def test_bit_exact(H, W, kind):
    rng = np.random.default_rng(H * 1000 + W)
    ref = rng.integers(0, 256, (H, W), dtype=np.uint8)
    cur = rng.integers(0, 256, (H, W), dtype=np.uint8)
    if kind == "moved":
        cur = np.roll(ref, (3, -8), (0, 1))
    elif kind == "flat":                       # every candidate ties: the lowest raster index
        cur[:], ref[:] = 70, 90
    plan = mb.merit_plan_sad(H, W, 16, 8)
    assert plan.launch_info()["kernel"] == "merit_sad_rowscan_pair<16,8>"
    sad, mv = mb.merit_sad_search(plan, torch.from_numpy(cur).cuda(), torch.from_numpy(ref).cuda())
    osad, omv = oracle.sad_search(cur, ref, 16, 8)
    assert np.array_equal(sad.cpu().numpy(), osad) and np.array_equal(mv.cpu().numpy(), omv)
