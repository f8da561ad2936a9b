"""Block matching with elimination by 4x4 sums (16x16 blocks): exact for any content, whichever way a block is decided."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


def _frames(kind, H, W, rng):
    yy, xx = np.mgrid[0:H, 0:W]
    smooth = 128 + 50 * np.sin(yy / 7.0 + 1) * np.cos(xx / 9.0) + 30 * np.sin((xx + 2 * yy) / 23.0)
    if kind == "moving":                  # few candidates left
        ref = smooth + rng.normal(0, 1.5, (H, W))
        cur = np.roll(smooth, (5, -9), (0, 1)) + rng.normal(0, 1.5, (H, W))
    elif kind == "noise":                 # never bounded
        ref, cur = rng.integers(0, 256, (2, H, W))
    elif isinstance(kind, tuple):         # ... with the blocks' matches at one displacement
        ref = rng.integers(0, 256, (H, W))
        cur = np.roll(ref, (-kind[0], -kind[1]), (0, 1))
    elif kind == "flat":                  # every candidate ties: the first in scan order
        ref = cur = np.full((H, W), 9)
    elif kind == "stripes":               # coarse, and many exact ties: too many candidates left
        ref = 255 * (yy // 8 % 2) + 0 * xx
        cur = np.roll(ref, 3, 0)
    elif kind == "checks":                # coarse, ties in both directions
        ref = 255 * ((yy // 4 + xx // 4) % 2)
        cur = np.roll(ref, (1, 2), (0, 1))
    else:                                 # "half": some blocks of a workgroup bounded, others not
        ref = np.where(xx % 48 < 20, smooth, 100) + rng.normal(0, 2, (H, W))
        cur = np.roll(ref, (-4, 3), (0, 1))
    return tuple(np.clip(np.round(f), 0, 255).astype(np.uint8) for f in (cur, ref))


@pytest.mark.parametrize("kind", ["moving", "noise", "flat", "stripes", "checks", "half"])
@pytest.mark.parametrize("H,W,R,blocks", [
    (16, 16, 32, 1), (16, 4, 32, 1),          # one block; fewer columns than a 16-byte load
    (17, 20, 32, 1), (50, 132, 32, 1),        # blocks past both edges
    (130, 130, 32, 1),                        # rows that are not whole dwords
    (17, 20, 32, 4), (50, 132, 32, 4),        # four blocks a workgroup, the last one ragged
    (128, 136, 32, 4), (130, 130, 32, 4),
    (50, 132, 16, 4), (130, 130, 16, 4),      # R = 16: fewer columns than lanes
    (130, 130, 16, 1), (17, 1030, 16, 1),     # ... one block a workgroup: from 64 blocks on
    (1030, 5, 16, 1), (260, 70, 16, 1),
])
def test_exact(kind, H, W, R, blocks):
    cur, ref = _frames(kind, H, W, np.random.default_rng(H * W + R))
    plan = mb.merit_plan_sad(H, W, 16, R)
    if blocks == 4:
        plan.set_tile((0, 4))
    li = plan.launch_info()
    print(kind, H, W, R, li, flush=True)
    assert li["kernel"] == "merit_sad_rowscan16<%d>" % R and li["tile"][1] == blocks
    _compare(plan, cur, ref, R)


def _compare(plan, cur, ref, R):
    sad, mv = mb.merit_sad_search(plan, torch.from_numpy(cur).cuda(), torch.from_numpy(ref).cuda())
    osad, omv = oracle.sad_search(cur, ref, 16, R)
    assert np.array_equal(sad.cpu().numpy(), osad) and np.array_equal(mv.cpu().numpy(), omv)
    return osad, omv


@pytest.mark.parametrize("dy", [-32, -1, 0, 1, 31, 32])
@pytest.mark.parametrize("dx", [-32, 31, 32])
@pytest.mark.parametrize("H,W,blocks", [(208, 208, 4), (210, 210, 4), (208, 208, 1)])
def test_matches_in_the_outer_columns_of_scanned_frames(dy, dx, H, W, blocks):
    """The 65th column is not a lane's: with four blocks a workgroup one wavefront takes it for all rows of a block."""
    cur, ref = _frames((dy, dx), H, W, np.random.default_rng(abs(dy * 100 + dx)))
    plan = mb.merit_plan_sad(H, W, 16, 32)
    if blocks == 4:
        plan.set_tile((0, 4))
    print(dy, dx, H, W, plan.launch_info(), flush=True)
    assert plan.launch_info()["tile"][1] == blocks
    osad, omv = _compare(plan, cur, ref, 32)
    assert (osad == 0).sum() >= 40 and (omv.reshape(-1, 2)[osad.ravel() == 0] == (dy, dx)).all()
