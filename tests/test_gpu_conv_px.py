"""1x1 layers on the matrix-product kernel (csrc/conv2d_px.hip) against the oracle: every tile with and without the added
tensor, planes and channel counts that are not whole 16-byte units, packed weights.  Bar: 2e-2*|r| + 1e-3 (fp16 products, fp32
accumulation, one rounding, against a double sum)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


CASES = [
    # N   Cin  H   W   Cout  residual
    (1, 16, 2, 4, 1, False),          # a single unit, a single step a quarter full
    (2, 24, 3, 3, 40, False),         # nine pixels: a unit and one cut
    (1, 17, 5, 7, 33, True),          # odd channels: rows of the weights on any 2-byte boundary
    (3, 65, 13, 9, 50, False),        # a second step of one channel
    (2, 130, 14, 14, 70, True),       # three steps, the last of two channels
    (1, 520, 11, 13, 96, False),      # nine steps: groups of four in flight and a remainder
    (1, 1000, 7, 7, 136, True),       # 49 pixels of a 64-pixel tile
    (2, 192, 31, 33, 130, False),
    (16, 64, 28, 28, 260, True),      # several tiles per compute unit
    (24, 72, 60, 20, 24, False),      # at most 32 output channels
    (5, 255, 57, 19, 64, False),      # rows of 255 channels
    (1, 248, 40, 41, 1000, False),
]

# One of each tile with a plane and channels that are not whole units, and one whose steps reach the loop that has the
# next ones in flight and leave a remainder (four steps ahead on the first two tiles, two or one on the others).
TILES = [
    # N   Cin  H   W   Cout  tile
    (3, 212, 12, 5, 1, (64, 32)),
    (2, 808, 3, 19, 1, (64, 32)),
    (17, 173, 2, 5, 585, (64, 64)),
    (11, 680, 3, 5, 827, (64, 64)),
    (17, 211, 3, 3, 981, (64, 128)),
    (21, 520, 6, 3, 1079, (64, 128)),
    (10, 129, 31, 52, 1, (128, 32)),
    (6, 520, 53, 26, 69, (128, 32)),
    (23, 130, 6, 23, 222, (128, 64)),
    (24, 544, 2, 33, 703, (128, 64)),
]


def _run(case, relu):
    N, Cin, H, W, Cout, residual = case
    rng = np.random.default_rng(Cin * 1000 + H * W)
    x = rng.standard_normal((N, Cin, H, W)).astype(np.float16)
    w = (rng.standard_normal((Cout, Cin, 1, 1)) / np.sqrt(Cin)).astype(np.float16)
    r = rng.standard_normal((N, Cout, H, W)).astype(np.float16)
    if residual:
        plan = mb.merit_plan_conv2d_residual(N, Cin, H, W, Cout, 1, 1, 1, 1, 0, 0, relu)
        ref = oracle.conv2d_residual(x, w, r, (1, 1), (0, 0), bool(relu))
    else:
        plan = (mb.merit_plan_conv2d_relu if relu else mb.merit_plan_conv2d)(N, Cin, H, W, Cout, 1, 1, 1, 1, 0, 0)
        ref = oracle.conv2d(x, w, (1, 1), (0, 0), relu=bool(relu))
    li = plan.launch_info()
    print(case, li, flush=True)
    assert li["block"][0] == 512 and li["kernel"] == "merit_conv2d_px"
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    dx, dw, dr = (torch.from_numpy(a).cuda() for a in (x, w, r))
    if residual:
        mb.merit_conv2d_residual(plan, dx, dw, dr, y)
    else:
        mb.merit_conv2d(plan, dx, dw, y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    got, ref = y.cpu().numpy().astype(np.float64), ref.astype(np.float64)
    assert np.all(np.abs(got - ref) <= 2e-2 * np.abs(ref) + 1e-3), np.abs(got - ref).max()
    return plan, dx, dw, dr, y


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("relu", [0, 1])
def test_against_the_oracle(case, relu):
    plan, dx, dw, dr, y = _run(case, relu)
    if case[5]:                       # the added tensor may be the output itself
        z = dr.clone()
        assert torch.equal(mb.merit_conv2d_residual(plan, dx, dw, z, z), y)
    elif case[1] % 8 == 0 and case[1] >= 32 and case[4] > 32:
        assert torch.equal(mb.merit_conv2d_packed(plan, dx, mb.merit_conv2d_pack_weights(plan, dw)), y)
        z = torch.empty_like(y)
        assert torch.equal(mb.merit_conv2d_packed_noalloc(plan, dx, dw, z), y)
    else:
        with pytest.raises(mb.MeritError):
            mb.merit_plan_packed_weights_bytes(plan)


@pytest.mark.parametrize("case", TILES)
@pytest.mark.parametrize("residual", [False, True])
def test_every_tile(case, residual):
    plan, dx, dw, dr, y = _run(case[:5] + (residual,), 0)
    (tm, tn), W = case[5], case[3]
    tile = plan.launch_info()["tile"]
    assert tile[1] == tn and tile[2] == -(-tm // W), tile


@pytest.mark.parametrize("Cin,H,W", [(33, 3, 5), (70, 9, 9), (100, 13, 9)])
def test_neighbouring_rows_do_not_leak(Cin, H, W):
    """What is loaded past a plane's or a weight row's end belongs to the next image or output channel."""
    x = torch.randn((2, Cin, H, W), device="cuda").half()
    w = torch.randn((40, Cin, 1, 1), device="cuda").half()
    x[1], w[7] = float("nan"), float("inf")
    y = mb.merit_conv2d(mb.merit_plan_conv2d(2, Cin, H, W, 40, 1, 1, 1, 1, 0, 0), x, w)
    keep = [c for c in range(40) if c != 7]
    assert bool(torch.isfinite(y[0, keep]).all()) and bool(torch.isnan(y[1]).all())
    assert not bool(torch.isfinite(y[0, 7]).any())
