"""Work lists near the limits of a launch (2^32 threads) and of the kernels' 32-bit divisions: the kernels that smaller calls
run on take them, in another form where that is what it takes."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb


def _threads(li):
    return li["grid"][0] * li["grid"][1] * li["grid"][2] * li["block"][0]


# N, H, W, k: a tile an image and 2^24 and more of them; tiles whose count a frame's height makes too large to divide by
SEP = [((1 << 24) + 3, 1, 4, 3), ((1 << 24) + 3, 1, 5, 3), ((1 << 24) + 3, 1, 1, 28), (1 << 24, 8, 8, 3),
       (1, 3200000, 8, 20), (45, 439354, 8, 25), (35338139, 2, 93, 26)]


@pytest.mark.parametrize("shape", SEP)
def test_separable_filters_of_many_tiles(shape):
    li = mb.merit_plan_sepfilter(*shape).launch_info()
    assert li["kernel"] == "merit_sepfilter_tile" and _threads(li) < 1 << 32, li


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SEP[0], SEP[1], SEP[4], ((1 << 24) + 3, 1, 4, 1), ((1 << 24) + 3, 1, 5, 9), ((1 << 24) + 3, 1, 4, 16)])
def test_separable_filters_of_many_tiles_against_the_oracle(shape):
    N, H, W, k = shape
    rng = np.random.default_rng(k)
    x = rng.integers(0, 256, (N, H, W), dtype=np.uint8).astype(np.float32)
    kx, ky = (rng.standard_normal(k).astype(np.float32) for _ in range(2))
    y = mb.merit_sepfilter(mb.merit_plan_sepfilter(*shape), *(torch.from_numpy(a).cuda() for a in (x, kx, ky))).cpu().numpy()
    # 2k fp32 multiply-adds of at most |kx| |ky| max|x|
    assert np.abs(y - oracle.sepfilter(x, kx, ky)).max() <= 1e-5 * np.abs(kx).sum() * np.abs(ky).sum() * 255


# 2x2 means of tall frames and long lists of planes: N, C, H, W
POOL = [(4, 64, 2158, 3838), (8, 1, 65536, 10), (13, 2656, 1996, 61), (348, 16674, 68, 31)]


@pytest.mark.parametrize("shape", POOL)
def test_pooling_of_long_lists_stays_on_its_kernel(shape):
    li = mb.merit_plan_pool2d(*shape, 2, 2, 2, 2, 0, 0, 1).launch_info()
    assert li["kernel"] == "merit_pool2d_lanes2_s2<avg,2>" and _threads(li) < 1 << 32, li


@pytest.mark.gpu
@pytest.mark.parametrize("avg", [False, True])
def test_pooling_of_long_lists_against_the_oracle(avg):
    x = np.random.default_rng(3).standard_normal((8, 1, 65536, 10)).astype(np.float32)
    y = mb.merit_pool2d(mb.merit_plan_pool2d(8, 1, 65536, 10, 2, 2, 2, 2, 0, 0, avg), torch.from_numpy(x).cuda()).cpu().numpy()
    ref = oracle.pool2d(x, (2, 2), (2, 2), (0, 0), "avg" if avg else "max")
    if avg:       # sums of four in another order
        assert np.all(np.abs(y - ref) <= 2.0 ** -22 * oracle.pool2d(np.abs(x), (2, 2), (2, 2), (0, 0), "avg"))
    else:
        assert np.array_equal(y, ref)


# depthwise layers with wide rows or many planes: N, C, H, W, k, s
DW = [(1, 3, 1400, 17000, 3, 2), (1, 3, 1400, 17000, 5, 2), (5, 63, 12, 19888, 3, 2), (4, 3, 923, 13451, 5, 2),
      (47, 8, 322, 4166, 3, 2), (2, 2400, 174, 1578, 3, 2), (30, 23, 13141, 7, 5, 2)]


@pytest.mark.parametrize("shape", DW)
def test_large_depthwise_layers_stay_on_the_kernel_without_lds(shape):
    N, C, H, W, k, s = shape
    li = mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, k // 2, k // 2).launch_info()
    assert li["kernel"] == "merit_dwconv_lanes" and _threads(li) < 1 << 32, li


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [DW[0], DW[3]])
def test_large_depthwise_layers_against_the_oracle(shape):
    N, C, H, W, k, s = shape
    rng = np.random.default_rng(k)
    x = rng.standard_normal((N, C, H, W), dtype=np.float32).astype(np.float16)
    w = (rng.standard_normal((C, k, k)) / k).astype(np.float16)
    plan = mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, k // 2, k // 2)
    y = mb.merit_conv2d_depthwise(plan, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()).cpu().numpy()
    ref = oracle.conv2d_depthwise(x, w, (s, s), (k // 2, k // 2)).astype(np.float64)
    mag = oracle.conv2d_depthwise(np.abs(x), np.abs(w), (s, s), (k // 2, k // 2)).astype(np.float64)
    # one rounding to binary16 on either side and k*k fp32 sums in another order
    assert np.all(np.abs(y - ref) <= 2.0 ** -10 * np.abs(ref) + k * k * 2.0 ** -23 * mag + 1e-7)


# 1x1 layers on millions of images: N, Cin, H, W, Cout
PX = [((1 << 23) + 1, 16, 1, 8, 40), (1 << 23, 40, 2, 8, 48), (5812858, 643, 1, 8, 399)]


@pytest.mark.parametrize("shape", PX)
def test_1x1_layers_on_millions_of_images(shape):
    li = mb.merit_plan_conv2d(*shape, 1, 1, 1, 1, 0, 0).launch_info()
    assert li["kernel"] in ("merit_conv2d_chws", "merit_conv2d_chblock", "merit_conv2d_chpass") and _threads(li) < 1 << 32, li


@pytest.mark.gpu
def test_1x1_layers_on_millions_of_images_against_the_oracle():
    N, Cin, H, W, Cout = PX[0]
    rng = np.random.default_rng(2)
    some = rng.standard_normal((1001, Cin, H, W)).astype(np.float16)        # the batch repeats these
    w = (rng.standard_normal((Cout, Cin, 1, 1)) / 4).astype(np.float16)
    x = torch.from_numpy(some).cuda()[torch.arange(N, device="cuda") % 1001]
    y = mb.merit_conv2d(mb.merit_plan_conv2d(N, Cin, H, W, Cout, 1, 1, 1, 1, 0, 0), x, torch.from_numpy(w).cuda())
    ref = torch.from_numpy(oracle.conv2d(some, w, (1, 1), (0, 0)).astype(np.float32)).cuda()
    mag = torch.from_numpy(oracle.conv2d(np.abs(some), np.abs(w), (1, 1), (0, 0)).astype(np.float32)).cuda()
    for i in range(0, N, 1001 * 1024):
        got = y[i:i + 1001 * 1024].float()
        j = torch.arange(i, i + len(got), device="cuda") % 1001
        # one rounding to binary16 on either side and fp32 sums of Cin products in another order
        assert bool(((got - ref[j]).abs() <= 2.0 ** -10 * ref[j].abs() + (Cin + 2) * 2.0 ** -23 * mag[j] + 1e-7).all())
