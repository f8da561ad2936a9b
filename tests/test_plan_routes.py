"""Which kernel a plan takes at the limits of what the kernels can hold, and what a plan accepts and refuses (no GPU)."""
import pytest

from paper_1911_03458_amd import binding as mb


def _conv(*shape):
    return mb.merit_plan_conv2d(*shape)


@pytest.mark.parametrize("shape", [
    (1, 4096, 1030, 256, 64, 3, 3, 1, 1, 1, 1),      # an image of 2.16 GB
    (1, 4000, 1080, 250, 64, 5, 5, 2, 2, 2, 2),
    (1, 3976, 1054, 256, 64, 3, 3, 1, 1, 1, 1),      # 2.146 GB, above 2 GiB with the last pass's padding channels
    (1, 4096, 16, 16, 30000, 3, 3, 1, 1, 1, 1),      # weights of 2.21 GB
])
def test_byte_offsets_of_the_multi_pass_kernel(shape):
    """merit_conv2d_chws addresses an image and the weights with byte offsets below 2 GiB: what is larger goes to a kernel
    with 64-bit addresses (a larger batch is several launches)."""
    assert _conv(*shape).launch_info()["kernel"] in ("merit_conv2d_chblock", "merit_conv2d_chpass")
    assert _conv(1, 3976, 1050, 256, 64, 3, 3, 1, 1, 1, 1).launch_info()["kernel"] == "merit_conv2d_chws"


def test_a_batch_may_be_larger_than_one_image():
    for shape in ((64, 100, 421, 421, 40, 3, 3, 1, 1, 1, 1), (64, 128, 400, 400, 72, 3, 3, 1, 1, 1, 1)):
        assert _conv(*shape).launch_info()["kernel"] == "merit_conv2d_chws"
