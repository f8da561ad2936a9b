"""8x8 blocks with a range of 4, seven blocks per wavefront and four block rows per workgroup: bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb


@pytest.mark.gpu
@pytest.mark.parametrize("H,W", [
    (8, 16), (8, 56), (64, 64), (40, 72),                               # few blocks: one workgroup, and a few
    (8, 521), (9, 528), (27, 168), (32, 224), (33, 169), (71, 75),      # whole and cut tiles of 4 x 7 blocks
    (300, 16), (279, 17), (301, 19), (270, 23),                         # the narrowest rows: every load crosses an edge
    (130, 120), (64, 75), (822, 1002),
])
def test_bit_exact(H, W):
    rng = np.random.default_rng(H * 1000 + W)
    ref = rng.integers(0, 256, (H, W), dtype=np.uint8)
    cur = np.roll(ref, (3, -4), (0, 1))
    cur[H // 2:] = rng.integers(0, 256, (H - H // 2, W), dtype=np.uint8)
    cur[:8, :8], ref[:12, :12] = 70, 90                      # a block whose candidates tie
    if W > 100:
        cur[:, 40:72], ref[:, 30:90] = 255, 0                # ... and the largest sums there are
    plan = mb.merit_plan_sad(H, W, 8, 4)
    li = plan.launch_info()
    assert li["kernel"] == "merit_sad_rowscan_seven" and li["grid"][0] == -(-H // 32) * -(-W // 56)
    n = plan.out_shape()[0] * plan.out_shape()[1]
    sad, mv = mb.merit_sad_search(plan, torch.from_numpy(cur).cuda(), torch.from_numpy(ref).cuda())
    osad, omv = oracle.sad_search(cur, ref, 8, 4)
    assert sad.numel() == n and np.array_equal(sad.cpu().numpy(), osad) and np.array_equal(mv.cpu().numpy(), omv)


def test_one_block_per_workgroup_on_request():
    plan = mb.merit_plan_sad(96, 128, 8, 4)
    assert plan.launch_info()["kernel"] == "merit_sad_rowscan_seven"
    plan.set_tile((0, 1))
    assert plan.launch_info()["kernel"] == "merit_sad_generic"
    assert mb.merit_plan_sad(96, 128, 8, 3).launch_info()["kernel"] == "merit_sad_generic"
