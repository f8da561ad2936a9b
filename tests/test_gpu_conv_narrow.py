"""Many-channel layers on the wave-specialised kernel whose input rows are not staged in 8-pixel units, against the oracle:
tall, narrow images (more staged rows than two such units per moving thread hold: units of 4 and 2 pixels) and rows of an
odd width where one-pixel units are faster.  Bar: 2e-2*|r| + 1e-3."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu

CASES = [
    # form       N  Cin  H    W  Cout k  sh sw ph pw  tile
    ("conv",     (3, 40, 138, 10, 72, 3, 3, 3, 3, 2, 1), None),            # 2-pixel units
    ("conv",     (2, 72, 129, 12, 40, 3, 3, 2, 4, 0, 0), None),            # 4-pixel units
    ("conv",     (2, 48, 91, 18, 74, 3, 3, 4, 4, 2, 1), None),
    ("conv",     (1, 128, 199, 6, 70, 3, 3, 2, 2, 0, 0), None),            # rows of fewer than 8 pixels
    ("conv",     (2, 88, 174, 4, 60, 3, 3, 4, 4, 1, 0), None),
    ("conv",     (2, 136, 141, 4, 70, 1, 1, 1, 4, 0, 1), None),            # 1x1, 64 channels per pass
    ("conv",     (2, 64, 160, 6, 256, 3, 3, 2, 2, 1, 1), (0, 0, 12, 64)),  # 12 wavefronts
    ("conv",     (2, 64, 150, 4, 256, 3, 3, 2, 2, 1, 1), (0, 0, 12, 64)),
    ("conv",     (2, 136, 5, 65, 40, 3, 3, 1, 1, 1, 1), None),             # odd widths, one-pixel units
    ("conv",     (2, 264, 9, 17, 72, 3, 3, 1, 1, 1, 1), None),
    ("conv",     (2, 256, 23, 21, 64, 3, 3, 2, 2, 1, 1), None),
    ("conv",     (2, 72, 7, 105, 100, 3, 3, 2, 2, 1, 1), None),
    ("residual", (2, 40, 151, 12, 77, 3, 3, 4, 4, 0, 1), None),
    ("pool",     (2, 24, 126, 12, 72, 3, 3, 6, 4, 2, 2), None),
]


@pytest.mark.parametrize("form,case,tile", CASES)
def test_against_the_oracle(form, case, tile):
    N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw = case
    rng = np.random.default_rng(Cin * 1000 + H)
    x = rng.standard_normal((N, Cin, H, W)).astype(np.float16)
    w = (rng.standard_normal((Cout, Cin, kh, kw)) / np.sqrt(Cin * kh * kw)).astype(np.float16)
    make = {"conv": mb.merit_plan_conv2d, "residual": mb.merit_plan_conv2d_residual, "pool": mb.merit_plan_conv2d_pool}
    plan = make[form](*case)
    if tile:
        plan.set_tile(tile)
    copies = 1                             # as many images as this kernel takes over at, the given ones repeated
    while plan.launch_info()["kernel"] == "merit_conv2d_split":
        copies *= 2
        plan = make[form](copies * N, *case[1:])
    print(form, case, plan.launch_info(), flush=True)
    assert plan.launch_info()["kernel"] == ("merit_conv2d_chws_pool" if form == "pool" else "merit_conv2d_chws")
    n = int(np.prod(plan.out_shape()))
    buf = torch.full((n + 128,), 777.0, dtype=torch.float16, device="cuda")
    y = buf[64:64 + n].view(plan.out_shape())
    xd, wd = torch.from_numpy(np.tile(x, (copies, 1, 1, 1))).cuda(), torch.from_numpy(w).cuda()
    if form == "residual":
        r = rng.standard_normal(plan.out_shape()).astype(np.float16)
        mb.merit_conv2d_residual(plan, xd, wd, torch.from_numpy(r).cuda(), y)
        ref = oracle.conv2d_residual(x, w, r, (sh, sw), (ph, pw), False)
    else:
        mb.merit_conv2d(plan, xd, wd, y)
        ref = (oracle.conv2d_pool if form == "pool" else oracle.conv2d)(x, w, (sh, sw), (ph, pw))
    assert bool((buf[:64] == 777).all()) and bool((buf[64 + n:] == 777).all())
    ref = np.tile(ref.astype(np.float64), (copies, 1, 1, 1))
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.abs(ref) + 1e-3)
    if form == "conv":
        assert torch.equal(mb.merit_conv2d_packed(plan, xd, mb.merit_conv2d_pack_weights(plan, wd)), y)
