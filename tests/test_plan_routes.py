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


@pytest.mark.parametrize("shape,tile", [
    ((3, 40, 138, 10, 72, 3, 3, 3, 3, 2, 1), None),
    ((64, 72, 129, 12, 40, 3, 3, 2, 4, 0, 0), None),       # (two images: the channels split among the wavefronts)
    ((2, 48, 91, 18, 74, 3, 3, 4, 4, 2, 1), None),
    ((1, 128, 199, 6, 70, 3, 3, 2, 2, 0, 0), None),
    ((2, 64, 150, 4, 256, 3, 3, 2, 2, 1, 1), (0, 0, 12, 64)),
    ((2, 64, 160, 6, 256, 3, 3, 2, 2, 1, 1), (0, 0, 12, 64)),
])
def test_narrow_layers_keep_the_multi_pass_kernel(shape, tile):
    """Many staged rows a tile: the kernel, its packed weights and its tile requests, whatever the width of its units."""
    plan = _conv(*shape)
    if tile:
        plan.set_tile(tile)
    assert plan.launch_info()["kernel"] == "merit_conv2d_chws"
    assert mb.merit_plan_packed_weights_bytes(plan) > 0


def test_narrow_layers_keep_the_fused_pooling():
    assert mb.merit_plan_conv2d_pool(2, 24, 126, 12, 72, 3, 3, 6, 4, 2, 2).launch_info()["kernel"] == "merit_conv2d_chws_pool"


def test_tiles_of_5x5_layers():
    """Two rounds of 256-pixel tiles (125 us) rather than three of 128-pixel tiles (156)."""
    li = _conv(9, 384, 63, 6, 734, 5, 5, 1, 1, 3, 3).launch_info()
    assert li["kernel"] == "merit_conv2d_chws" and li["tile"][1] == 64 and li["tile"][2] == 33      # rows of 8 pixels


def test_tiles_of_wide_odd_rows_with_a_stride():
    """One round of 64-channel tiles (13.9 us) rather than two of 32-channel ones (21.8)."""
    li = _conv(12, 80, 6, 123, 352, 3, 3, 2, 2, 1, 1).launch_info()
    assert li["kernel"] == "merit_conv2d_chws" and li["tile"][1] == 64


@pytest.mark.parametrize("shape", [
    (6, 1192, 83, 13, 381, 3, 3, 2, 2, 1, 1),       # 64-channel tiles 7.9 MiB, 32-channel ones 8.02
    (8, 336, 17, 102, 1344, 3, 3, 2, 2, 1, 1),      # ... 128-channel ones 8.12
    (5, 2824, 123, 63, 1431, 1, 1, 3, 3, 0, 0),     # passes of 16 channels 7.95 MiB, of 64 channels 8.3
    (4, 3632, 36, 110, 1079, 1, 1, 1, 1, 0, 0),     # weights of 7.5 MiB, read as they lie
])
def test_the_fixed_buffer_takes_the_smallest_packed_copy(shape):
    """A layer is not refused because the tiling that runs it pads its weights past the buffer."""
    plan = _conv(*shape)
    assert mb.merit_plan_packed_weights_bytes(plan) > mb.MERIT_NOALLOC_SCRATCH_BYTES
    accepted = mb.lib().merit_conv2d_packed_noalloc(plan.handle, None, None, None, None)       # (nothing is launched)
    assert accepted == mb.MERIT_ERR_NULL
    too_large = _conv(1, 1024, 16, 16, 1024, 3, 3, 1, 1, 1, 1)
    assert mb.lib().merit_conv2d_packed_noalloc(too_large.handle, None, None, None, None) == mb.MERIT_ERR_SCRATCH_LIMIT


@pytest.mark.parametrize("shape", [(1, 184, 60, 36, 3, 1), (1, 32, 17, 41, 4, 1), (1, 8, 16, 20, 2, 1)])
def test_correlation_off_the_multiple_of_8_refuses_tile_requests(shape):
    """Whichever kernel runs it: there is nothing to choose, and no request is accepted without effect."""
    plan = mb.merit_plan_correlation(*shape)
    before = plan.launch_info()
    for tile in ((0, 4), (1, 1, 1, 1), (0, 0, 4, 32)):
        with pytest.raises(mb.MeritError) as e:
            plan.set_tile(tile)
        assert e.value.status == mb.MERIT_ERR_UNSUPPORTED
    plan.set_tile((0,))                                     # no request: accepted
    assert plan.launch_info() == before


def test_launch_info_names_the_kernel_that_runs():
    """1x1 layers at stride 1, with and without a packed form; a tile request names the other kernel."""
    for make in (mb.merit_plan_conv2d, mb.merit_plan_conv2d_relu):
        plan = make(8, 256, 14, 14, 1024, 1, 1, 1, 1, 0, 0)
        assert plan.launch_info()["kernel"] == "merit_conv2d_px" and mb.merit_plan_packed_weights_bytes(plan) > 0
        plan.set_tile((0, 0, 8, 64))
        assert plan.launch_info()["kernel"] == "merit_conv2d_chws" and mb.merit_plan_packed_weights_bytes(plan) > 0
    assert mb.merit_plan_conv2d_residual(8, 256, 14, 14, 1024, 1, 1, 1, 1, 0, 0).launch_info()["kernel"] == "merit_conv2d_px"
    assert _conv(8, 256, 14, 14, 1024, 1, 1, 2, 2, 0, 0).launch_info()["kernel"] == "merit_conv2d_chws"


@pytest.mark.parametrize("shape,kernel", [
    ((1, 24, 9, 14, 3, 3, 2, 2, 1, 1), "merit_dwconv_lanes"),       # 2.8 us on the kernel for any window, 2.7 on this
    ((2, 40, 8, 17, 5, 5, 1, 1, 2, 2), "merit_dwconv_tile"),        # 3.5, 3.7 on the other: an odd width
    ((6, 56, 29, 8, 3, 3, 2, 2, 1, 1), "merit_dwconv_lanes"),       # 3.1, 2.8
    ((12, 144, 94, 24, 5, 5, 1, 1, 2, 2), "merit_dwconv_lanes"),    # 26.8, 7.8
    ((32, 512, 14, 14, 3, 3, 1, 1, 1, 1), "merit_dwconv_lanes"),    # 20.5, 6.8
    ((1, 8, 8, 4096, 3, 3, 1, 1, 0, 0), "merit_dwconv_lanes"),
    ((8, 10, 26, 2, 5, 5, 1, 1, 2, 2), "merit_dwconv_tile"),        # 3.5, 4.1 on the other
    ((1, 95, 29, 1, 5, 5, 2, 2, 2, 2), "merit_dwconv_tile"),        # 3.5, 4.2
])
def test_depthwise_layers_take_the_faster_kernel(shape, kernel):
    assert mb.merit_plan_conv2d_depthwise(*shape).launch_info()["kernel"] == kernel


@pytest.mark.parametrize("shape", [
    (0, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1), (0, 16, 12, 20, 64, 3, 3, 1, 1, 1, 1), (0, 256, 56, 56, 256, 3, 3, 1, 1, 1, 1),
    (0, 3, 64, 64, 64, 7, 7, 2, 2, 3, 3),
])
def test_fused_pooling_of_an_empty_batch(shape):
    plan = mb.merit_plan_conv2d_pool(*shape)
    assert plan.out_shape()[0] == 0 and plan.launch_info()["grid"][0] == 0
    assert mb.lib().merit_conv2d(plan.handle, None, None, None, None) == mb.MERIT_OK


@pytest.mark.parametrize("shape,tile", [
    ((2, 1024, 18, 18, 512, 3, 3, 1, 1, 1, 1), None),                 # the unfused layer splits the channels among the wavefronts
    ((1, 552, 50, 92, 88, 3, 3, 1, 1, 1, 1), None),
    ((1, 536, 96, 26, 416, 3, 3, 1, 1, 1, 1), (0, 0, 8, 32)),
    ((4, 256, 40, 56, 256, 3, 3, 1, 1, 1, 1), (0, 0, 8, 64)),
])
def test_launch_info_of_pooling_in_two_launches_is_the_multi_pass_kernels(shape, tile):
    """Its convolution sums in the order of the fused form, whatever the unfused layer's own plan takes; the figures are of
    the launch that runs: 128 or 256 pixels x a multiple of 32 channels."""
    N, Cin, H, W, Cout = shape[:5]
    li = mb.merit_plan_conv2d_pool(*shape).launch_info()
    assert li["kernel"] == "merit_conv2d_chws+merit_maxpool_f16"
    unfused = _conv(*shape)
    if tile:
        unfused.set_tile(tile)
        u = unfused.launch_info()
        assert (li["grid"][0], li["lds_bytes"], li["tile"][1]) == (u["grid"][0], u["lds_bytes"], u["tile"][1])
    blocks = -(-Cout // li["tile"][1])
    assert li["grid"][0] in [min(256, N * -(-H * W // m) * blocks) for m in (128, 256)] and li["tile"][3] == W


def test_tile_requests_of_block_matching():
    """What the header says of each request, and of the reported tile beside it."""
    def kernels(block, search, shape=(480, 640)):
        out = []
        for request in (None, 1, 4, 8, 2):
            plan = mb.merit_plan_sad(*shape, block, search)
            if request:
                plan.set_tile((0, request))
            li = plan.launch_info()
            out.append((li["kernel"].replace("merit_sad_", ""), li["tile"][1]))
        return out
    assert kernels(16, 32) == [("rowscan16<32>", 1), ("generic", 1)] + 3 * [("rowscan16<32>", 4)]
    assert kernels(16, 16) == [("rowscan16<16>", 1), ("generic", 1), ("rowscan16<16>", 4)] + 2 * [("rowscan_pair<16,16>", 8)]
    assert kernels(16, 8) == [("rowscan_pair<16,8>", 8), ("generic", 1), ("generic", 1)] + 2 * [("rowscan_pair<16,8>", 8)]
    assert kernels(8, 16) == [("rowscan_pair<8,16>", 8), ("generic", 1), ("generic", 1)] + 2 * [("rowscan_pair<8,16>", 8)]
    assert kernels(8, 4) == [("rowscan_seven", 7), ("generic", 1)] + 3 * [("rowscan_seven", 7)]
    assert kernels(16, 32, (2160, 3840))[0] == ("rowscan16<32>", 4) and kernels(12, 5)[0] == ("generic", 1)
