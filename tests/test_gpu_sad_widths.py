"""Block matching on frames whose rows are not whole dwords, on the row-scan kernels: bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(130, 129), (130, 130), (131, 131), (64, 270), (16, 1022), (1024, 10)])
@pytest.mark.parametrize("B,R", [(16, 32), (16, 16), (16, 8), (8, 16), (8, 8)])
def test_bit_exact(H, W, B, R):
    if -(-H // B) * -(-W // B) < 64:
        pytest.skip("the kernel for any shape takes the smallest frames")
    rng = np.random.default_rng(H * 1000 + W + R)
    ref = rng.integers(0, 256, (H, W), dtype=np.uint8)
    cur = np.roll(ref, (R // 2, -R), (0, 1))
    cur[H // 2:] = rng.integers(0, 256, (H - H // 2, W), dtype=np.uint8)
    cur[:B, :B], ref[:B + R, :B + R] = 70, 90                # a block where many candidates tie
    plan = mb.merit_plan_sad(H, W, B, R)
    assert "rowscan" in plan.launch_info()["kernel"]
    sad, mv = mb.merit_sad_search(plan, torch.from_numpy(cur).cuda(), torch.from_numpy(ref).cuda())
    osad, omv = oracle.sad_search(cur, ref, B, R)
    assert np.array_equal(sad.cpu().numpy(), osad) and np.array_equal(mv.cpu().numpy(), omv)
