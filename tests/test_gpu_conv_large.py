"""Many-channel layers on batches of more than 2 GiB: every image as in a small batch, the first ones' padding rows
above all (byte offsets past the end of a descriptor are how the kernel gets its zeros)."""
import pytest
import torch

from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Cin,H,W,Cout,form", [
    (64, 100, 421, 421, 40, "raw"),           # odd planes: the second launch starts at an even image
    (64, 128, 400, 400, 72, "raw"),
    (64, 128, 400, 400, 72, "packed"),
    (64, 128, 400, 400, 64, "residual"),
    (1090, 64, 126, 124, 64, "pool"),
])
def test_images_of_a_large_batch(N, Cin, H, W, Cout, form):
    def plan(n):
        args = (n, Cin, H, W, Cout, 3, 3, 1, 1, 1, 1)
        make = {"residual": mb.merit_plan_conv2d_residual, "pool": mb.merit_plan_conv2d_pool}
        p = make.get(form, mb.merit_plan_conv2d)(*args)
        assert p.launch_info()["kernel"].startswith("merit_conv2d_chws")
        return p

    def run(p, x, r):
        if form == "packed":
            return mb.merit_conv2d_packed(p, x, mb.merit_conv2d_pack_weights(p, w))
        return mb.merit_conv2d_residual(p, x, w, r) if form == "residual" else mb.merit_conv2d(p, x, w)

    torch.manual_seed(N + Cin)
    x = torch.randn((N, Cin, H, W), device="cuda", dtype=torch.float16)
    assert x.numel() * 2 > 2 ** 31
    w = torch.randn((Cout, Cin, 3, 3), device="cuda", dtype=torch.float16) * 0.03
    r = torch.randn((N, Cout, H, W), device="cuda", dtype=torch.float16) if form == "residual" else None
    y = run(plan(N), x, r)
    small = plan(2)
    for i in (0, 1, N // 2, N - 2):
        want = run(small, x[i:i + 2].clone(), r[i:i + 2].clone() if r is not None else None)
        assert torch.equal(y[i:i + 2], want), i     # (the order of a sum does not depend on the tiling)
