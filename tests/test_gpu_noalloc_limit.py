"""Layers whose packed weights fit the library's fixed buffer on another tiling than the one that runs them: the same
bits through either."""
import pytest
import torch

from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 1192, 83, 13, 381, 3, 3, 2, 2, 1, 1),
    (5, 2824, 123, 63, 1431, 1, 1, 3, 3, 0, 0),
    (1, 3632, 36, 110, 1079, 1, 1, 1, 1, 0, 0),
])
def test_same_bits(shape):
    N, Cin, H, W, Cout, kh, kw = shape[:7]
    torch.manual_seed(Cin)
    x = torch.randn((N, Cin, H, W), device="cuda").half()
    w = (torch.randn((Cout, Cin, kh, kw), device="cuda") / (Cin * kh * kw) ** 0.5).half()
    plan = mb.merit_plan_conv2d(*shape)
    print(shape, plan.launch_info(), mb.merit_plan_packed_weights_bytes(plan), flush=True)
    assert mb.merit_plan_packed_weights_bytes(plan) > mb.MERIT_NOALLOC_SCRATCH_BYTES
    y = torch.full(plan.out_shape(), 7.0, dtype=torch.float16, device="cuda")
    mb.merit_conv2d_packed_noalloc(plan, x, w, y)
    assert torch.equal(y, mb.merit_conv2d(plan, x, w))
    assert torch.equal(y, mb.merit_conv2d_packed(plan, x, mb.merit_conv2d_pack_weights(plan, w)))
