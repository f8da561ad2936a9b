"""1x1 layers whose planes and channels the 16-byte units of eight do not divide, on every tile, against the oracle; the added
tensor may be the output, so that no pixel may be stored by two threads there."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu

CASES = [
    # N  Cin  H   W   Cout
    (2, 16, 2, 4, 8),          # one unit a plane, one short step
    (3, 17, 3, 3, 33),         # nine pixels: two units that share seven
    (2, 63, 5, 13, 40),        # 65 pixels: the second tile is one pixel
    (2, 64, 3, 43, 70),        # 129 pixels, one whole step
    (1, 71, 11, 13, 96),       # a step and a cut unit
    (2, 191, 9, 15, 64),
    (1, 303, 25, 27, 272),     # more than 256 channels, not a multiple of 8
    (2, 1029, 3, 11, 130),
    (24, 248, 7, 18, 992),     # 128 x 128 tiles
    (25, 130, 53, 19, 520),
    (1, 260, 8, 16, 128),      # whole tiles, channels off the 8
    (8, 260, 56, 56, 64),
    (3, 1028, 16, 16, 40),
    (17, 173, 2, 5, 585),      # 64 x 64 tiles
    (17, 211, 3, 3, 981),      # 64 x 128
    (23, 130, 6, 23, 222),     # 128 x 64
]


def _tile(li, W):
    return next(t for t in (64, 128) if -(-t // W) == li["tile"][2]), li["tile"][1]


@pytest.mark.parametrize("make", [mb.merit_plan_conv2d, mb.merit_plan_conv2d_residual])
def test_the_cases_reach_every_tile(make):
    tiles = {_tile(make(N, Cin, H, W, Cout, 1, 1, 1, 1, 0, 0).launch_info(), W) for N, Cin, H, W, Cout in CASES}
    assert tiles == {(64, 32), (64, 64), (64, 128), (128, 32), (128, 64), (128, 128)}


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_cut_units(case, residual):
    N, Cin, H, W, Cout = case
    rng = np.random.default_rng(Cin + W)
    x = rng.standard_normal((N, Cin, H, W)).astype(np.float16)
    w = (rng.standard_normal((Cout, Cin, 1, 1)) / np.sqrt(Cin)).astype(np.float16)
    r = rng.standard_normal((N, Cout, H, W)).astype(np.float16)
    make = mb.merit_plan_conv2d_residual if residual else mb.merit_plan_conv2d
    plan = make(N, Cin, H, W, Cout, 1, 1, 1, 1, 0, 0)
    assert plan.launch_info()["kernel"] == "merit_conv2d_px"
    n = N * Cout * H * W
    buf = torch.full((n + 128,), 777.0, device="cuda", dtype=torch.float16)
    y = buf[64:64 + n].view(N, Cout, H, W)
    dx, dw = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    if residual:
        y.copy_(torch.from_numpy(r))
        mb.merit_conv2d_residual(plan, dx, dw, y, y)
        ref = oracle.conv2d_residual(x, w, r, (1, 1), (0, 0), False)
    else:
        mb.merit_conv2d(plan, dx, dw, y)
        ref = oracle.conv2d(x, w, (1, 1), (0, 0))
    assert bool((buf[:64] == 777).all()) and bool((buf[-64:] == 777).all())
    # one rounding to binary16 (2^-11) and fp32 sums of Cin products in another order (at most Cin 2^-24 of their magnitudes)
    ref = ref.astype(np.float64)
    mag = oracle.conv2d(np.abs(x), np.abs(w), (1, 1), (0, 0)).astype(np.float64) + np.abs(r) * residual
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 2.0 ** -10 * np.abs(ref) + (Cin + 2) * 2.0 ** -23 * mag + 1e-7)
