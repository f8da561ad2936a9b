"""Many-channel layers on few pixels: the kernel that splits the channels among the wavefronts."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu

CASES = [
    # N, Cin, H, W, Cout, k, s, p, dilation; pixels of a tile, columns of a rectangular one (0: a run of adjacent pixels)
    ((2, 17, 5, 9, 33, 3, 1, 1, 1), (32, 0)),            # two slices, the second of one channel
    ((1, 24, 4, 9, 40, 3, 1, 1, 1), (32, 0)),            # the second slice half a slice
    ((2, 56, 4, 8, 64, 3, 1, 1, 1), (32, 0)),            # one unit per row, one tile of exactly 32 pixels
    ((1, 136, 11, 3, 33, 3, 1, 1, 1), (32, 0)),          # a tile of one pixel; nine slices
    ((3, 129, 9, 13, 65, 3, 1, 1, 1), (32, 0)),          # ... of one channel; 13-pixel rows: the last unit overlaps
    ((2, 264, 7, 7, 40, 3, 1, 1, 1), (32, 0)),           # 7x7 planes: loads moved at the last channel's end
    ((2, 64, 12, 40, 48, 3, 2, 1, 1), (32, 0)),          # stride 2
    ((1, 80, 14, 47, 40, 3, 1, 2, 2), (32, 8)),          # dilated window, odd rows, two units per lane
    ((2, 72, 30, 64, 40, 3, 1, 0, 1), (32, 0)),          # no padding
    ((1, 256, 14, 14, 96, 3, 1, 1, 1), (32, 0)),
    ((4, 256, 14, 14, 256, 3, 1, 1, 1), (32, 0)),        # weights larger than the images: the list by channel block
    ((1, 32, 5, 5, 40, 5, 1, 2, 1), (32, 0)),            # 5x5
    ((2, 37, 9, 10, 36, 5, 2, 2, 1), (32, 0)),
    ((1, 144, 21, 23, 56, 5, 1, 2, 1), (32, 0)),
    # rectangular tiles: rows too long to be staged whole
    ((1, 40, 9, 95, 40, 5, 2, 2, 1), (32, 8)),           # 48 columns: a cut tile beside whole ones, the last unit moved back
    ((2, 72, 11, 111, 33, 3, 2, 1, 1), (32, 16)),        # 56 columns, six rows
    ((1, 88, 5, 130, 40, 3, 1, 1, 1), (32, 8)),          # two columns in the last tile
    ((2, 49, 7, 97, 24, 3, 2, 0, 1), (32, 8)),           # channels off the multiple of 8, no padding
    ((1, 80, 12, 150, 40, 3, 1, 2, 2), (32, 8)),         # dilated window
    ((2, 32, 7, 50, 27, 3, 2, 1, 1), (32, 32)),          # 32 columns
    ((4, 80, 5, 39, 22, 5, 2, 2, 1), (32, 32)),
    ((12, 36, 5, 149, 68, 3, 2, 1, 1), (32, 8)),         # more workgroups than compute units
    ((2, 38, 20, 10, 31, 3, 2, 1, 1), (32, 0)),          # two units per lane
    ((2, 29, 3, 33, 28, 5, 2, 2, 1), (32, 0)),
    ((1, 56, 4, 34, 53, 5, 2, 2, 1), (32, 0)),
    ((1, 64, 4, 6, 48, 5, 2, 2, 1), (32, 0)),            # 5x5 on rows of fewer than 8 pixels
    # 64-pixel tiles
    ((9, 264, 7, 7, 480, 3, 1, 1, 1), (64, 0)),          # rows of fewer than 8 pixels; the list by channel block
    ((9, 40, 12, 5, 480, 3, 1, 1, 1), (64, 0)),
    ((8, 256, 14, 14, 256, 3, 1, 1, 1), (64, 0)),
    ((19, 32, 22, 9, 33, 3, 1, 1, 1), (64, 0)),          # the list by tile
    ((22, 17, 10, 13, 200, 3, 2, 1, 1), (64, 0)),        # channels off the multiple of 8
    ((20, 32, 9, 20, 200, 3, 2, 1, 1), (64, 0)),         # two units per lane
    ((15, 19, 5, 62, 35, 3, 1, 1, 1), (64, 8)),          # rectangles of 8, 16 and 32 columns
    ((22, 19, 3, 130, 22, 3, 1, 1, 1), (64, 16)),
    ((12, 19, 10, 62, 40, 3, 1, 1, 1), (64, 32)),
    ((18, 40, 6, 143, 104, 3, 2, 1, 1), (64, 16)),       # more workgroups than compute units
    ((12, 24, 7, 7, 360, 5, 1, 2, 1), (64, 0)),          # 5x5
    ((16, 45, 7, 9, 300, 5, 1, 2, 1), (64, 0)),
    ((22, 104, 12, 12, 256, 5, 2, 2, 1), (64, 0)),       # the list by channel block
    ((22, 32, 12, 14, 39, 5, 1, 2, 1), (64, 0)),         # the list by tile
    ((5, 18, 25, 35, 34, 5, 1, 2, 1), (64, 8)),          # rectangles
    ((19, 32, 6, 141, 39, 5, 2, 2, 1), (64, 16)),
    ((8, 24, 40, 36, 68, 5, 2, 2, 1), (64, 32)),
    ((11, 32, 15, 108, 175, 5, 2, 2, 1), (64, 8)),       # more workgroups than compute units
]


@pytest.mark.parametrize("case,tile", CASES)
def test_against_the_oracle_raw_and_packed(case, tile):
    N, Cin, H, W, Cout, k, s, p, d = case
    rng = np.random.default_rng(Cin * 1000 + W)
    x = rng.standard_normal((N, Cin, H, W)).astype(np.float16)
    w = (rng.standard_normal((Cout, Cin, k, k)) / np.sqrt(Cin * k * k)).astype(np.float16)
    plan = mb.merit_plan_conv2d_dilated(N, Cin, H, W, Cout, k, k, s, s, p, p, d, d, 1)
    li = plan.launch_info()
    print(case, li, flush=True)
    (oh, ow), (pixels, columns) = plan.out_shape()[2:], tile
    assert li["kernel"] == "merit_conv2d_split" and li["tile"][1] == 32 and li["tile"][3] == (columns or ow)
    tiles = -(-oh // (pixels // columns)) * -(-ow // columns) if columns else -(-oh * ow // pixels)
    assert li["grid"][0] == N * -(-Cout // 32) * tiles
    # no numbers beside the operands: what is loaded past a row, an image or the weights must not reach a sum
    xb = torch.full((x.size + 256,), float("nan"), dtype=torch.float16, device="cuda")
    wb = torch.full((w.size + 256,), float("inf"), dtype=torch.float16, device="cuda")
    xb[128:-128], wb[128:-128] = torch.from_numpy(x).flatten(), torch.from_numpy(w).flatten()
    xd, wd = xb[128:-128].view(x.shape), wb[128:-128].view(w.shape)
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    mb.merit_conv2d(plan, xd, wd, y)
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = oracle.conv2d(x, w, (s, s), (p, p), relu=True, dilation=(d, d)).astype(np.float64)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.abs(ref) + 1e-3)
    if Cin % 8 == 0 and Cin >= 32 and Cout > 32:
        assert torch.equal(mb.merit_conv2d_packed(plan, xd, mb.merit_conv2d_pack_weights(plan, wd)), y)


def test_an_image_or_an_output_channel_without_numbers_stays_alone():
    """NaN in one image, infinities in one output channel's weights: the others are what they are without them (the last
    slice and the channel blocks are padded with zeros, not with neighbours)."""
    N, Cin, H, W, Cout = 3, 24, 7, 9, 40
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal((N, Cin, H, W)).astype(np.float16)).cuda()
    w = torch.from_numpy((rng.standard_normal((Cout, Cin, 3, 3)) / 15).astype(np.float16)).cuda()
    plan = mb.merit_plan_conv2d(N, Cin, H, W, Cout, 3, 3, 1, 1, 1, 1)
    clean = mb.merit_conv2d(plan, x, w)
    x[1], w[7] = float("nan"), float("inf")
    y = mb.merit_conv2d(plan, x, w)
    keep = [c for c in range(Cout) if c != 7]
    assert torch.equal(y[[0, 2]][:, keep], clean[[0, 2]][:, keep])
    assert not bool(torch.isfinite(y[:, 7]).any())
