"""Many-channel layers on channel counts, output channels and row widths that are not whole units, on the
wave-specialised kernel and on whatever the plan of so few images takes, against the oracle.  Bar: 2e-2*|r| + 1e-3."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


CASES = [
    # N  Cin  H   W  Cout k  s   kernel of a plan without an added tensor
    (2, 17, 9, 8, 33, 3, 1, "chws"),           # a group of one channel, rows of one whole unit
    (2, 41, 11, 9, 24, 3, 1, "split"),         # rows of a unit and one pixel; at most 32 output channels
    (3, 23, 17, 15, 70, 3, 2, "split"),        # seven of eight channels, stride 2
    (2, 100, 14, 14, 96, 3, 1, "split"),
    (2, 165, 12, 110, 60, 3, 2, "split"),      # wide rows, two units per moving thread
    (2, 31, 30, 56, 128, 3, 1, "chws"),
    (2, 272, 13, 9, 24, 3, 1, "split"),
    (2, 24, 19, 51, 264, 3, 1, "chws"),
    (2, 65, 12, 10, 40, 5, 1, "split"),        # 5x5
    (2, 36, 21, 27, 17, 5, 2, "split"),
    (3, 50, 31, 30, 56, 1, 2, "chws"),         # 1x1 at stride 2
    (2, 40, 13, 7, 40, 3, 1, "split"),         # rows of fewer than 8 pixels: one-pixel units
    (2, 52, 24, 28, 64, 5, 1, "split"),        # 5x5 on 128-pixel tiles, 64 and 32 channels
    (2, 128, 14, 15, 96, 5, 2, "split"),
    (2, 16, 11, 13, 40, 3, 1, "chws"),         # 16 channels on rows off the 8 pixels
    (3, 16, 8, 16, 24, 5, 1, "chws"),          # ... and with 5x5 windows on any row
    (2, 32, 12, 15, 32, 3, 2, "split"),        # at most 32 output channels, likewise
    (2, 64, 9, 10, 24, 3, 1, "split"),
    (2, 24, 8, 32, 24, 5, 2, "chws"),
]


@pytest.mark.parametrize("form,case", [(form, c) for form in ("plain", "residual") for c in CASES] +
                         [("multi-pass", c) for c in CASES if c[-1] == "split"])
def test_against_the_oracle(form, case):
    N, Cin, H, W, Cout, k, s, planned = case
    residual = form == "residual"
    args = (Cin, H, W, Cout, k, k, s, s, k // 2, k // 2)
    rng = np.random.default_rng(Cin * 1000 + W)
    x = rng.standard_normal((N, Cin, H, W)).astype(np.float16)
    w = (rng.standard_normal((Cout, Cin, k, k)) / np.sqrt(Cin * k * k)).astype(np.float16)
    plan = mb.merit_plan_conv2d_residual(N, *args, 1) if residual else mb.merit_plan_conv2d_relu(N, *args)
    if form == "multi-pass":               # as many images as that kernel takes over at, the given ones repeated
        copies = 1
        while plan.launch_info()["kernel"] == "merit_conv2d_split":
            copies *= 2
            plan = mb.merit_plan_conv2d_relu(copies * N, *args)
        x = np.tile(x, (copies, 1, 1, 1))
    kernel = plan.launch_info()["kernel"]
    print(case, plan.launch_info(), flush=True)
    if form == "plain":
        assert kernel == "merit_conv2d_" + planned
    elif not residual or k == 3:           # (with an added tensor: 3x3 windows, and 1x1 from 128 channels on)
        assert kernel == "merit_conv2d_chws"
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    r = rng.standard_normal(plan.out_shape()).astype(np.float16)
    # the images and output channels next to the ones that are compared hold no numbers: what is loaded past a row
    # of pixels or of weights must not leak
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    xd[1], wd[3] = float("nan"), float("inf")
    if residual:
        mb.merit_conv2d_residual(plan, xd, wd, torch.from_numpy(r).cuda(), y)
        ref = oracle.conv2d_residual(x, w, r, (s, s), (k // 2, k // 2), True)
    else:
        mb.merit_conv2d(plan, xd, wd, y)
        ref = np.tile(oracle.conv2d(x[:N], w, (s, s), (k // 2, k // 2), relu=True), (len(x) // N, 1, 1, 1))
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    keep = [c for c in range(Cout) if c != 3]
    imgs = [i for i in range(len(x)) if i != 1]
    got, ref = y.cpu().numpy().astype(np.float64)[imgs][:, keep], ref.astype(np.float64)[imgs][:, keep]
    assert np.all(np.abs(got - ref) <= 2e-2 * np.abs(ref) + 1e-3), np.abs(got - ref).max()
    if residual:
        return
    if Cin % 8 == 0 and Cin >= 32 and Cout > 32:
        assert torch.equal(mb.merit_conv2d_packed(plan, xd, mb.merit_conv2d_pack_weights(plan, wd))[imgs][:, keep], y[imgs][:, keep])
    else:                                                # (no packed form on these counts)
        with pytest.raises(mb.MeritError) as e:
            mb.merit_plan_packed_weights_bytes(plan)
        assert e.value.status == mb.MERIT_ERR_UNSUPPORTED
