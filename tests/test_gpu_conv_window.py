"""The window kernel (unit stride, output grid = input grid, the tile's pixels and what their taps reach in LDS): against the oracle at the
edges of its windows, tiles and images, in every form the fused calls take, and which layers the planner gives to it."""
import pytest
import torch

from paper_1807_11205_amd import api, inputs

WIDE, NARROW = (256, 128, 64, 8, 19), (256, 64, 64, 4, 19)      # tile, k tile, wavefronts, 16 + depth of the filter's ring


def plan(op, *a):
    return api.jz_conv2d_describe_plan(op, api.conv_desc(*a))


def test_which_layers_run_on_it():
    for op in (api.JZ_FWD, api.JZ_BWD_DATA):
        assert "replaced by window tile 256x64x64, 4 wavefronts, ring 19" in plan(op, 64, 56, 56, 64, 64, 3, 3, 1, 1)
        assert "replaced by window tile 256x128x64, 8 wavefronts, ring 19" in plan(op, 64, 28, 28, 128, 128, 3, 3, 1, 1)
        for other in [(64, 64, 64, 64, 64, 3, 3, 1, 1),        # 256 pixels and what their taps reach: 386 of 384 rows
                      (64, 56, 56, 64, 64, 3, 3, 2, 1), (64, 56, 56, 64, 64, 3, 3, 1, 0), (64, 56, 56, 64, 64, 1, 1, 1, 0),
                      (64, 28, 28, 96, 96, 3, 3, 1, 1), (1, 28, 28, 64, 64, 3, 3, 1, 1), (64, 27, 27, 64, 64, 7, 7, 1, 3)]:
            assert "window" not in plan(op, *other), other
            with pytest.raises(RuntimeError):
                api.jz_conv2d_tune_set(op, api.conv_desc(*other[:3], 96, 96, *other[5:]), *NARROW, 1)
    assert "window" not in plan(api.JZ_BWD_WEIGHT, 64, 56, 56, 64, 64, 3, 3, 1, 1)


def test_offsets_within_a_window_have_31_bits():
    """384 rows of so many channels; the tensors themselves (3 x 3 pixels, eight filters) are below the 4 GB that a descriptor reaches."""
    for op, at in ((api.JZ_FWD, 3), (api.JZ_BWD_DATA, 4)):
        d = [1, 3, 3, 8, 8, 3, 3, 1, 1]
        d[at] = (1 << 31) // 768 // 64 * 64
        api.jz_conv2d_tune_set(op, api.conv_desc(*d), *WIDE, 1)
        api.jz_conv2d_tune_clear()
        d[at] += 64
        with pytest.raises(RuntimeError):
            api.jz_conv2d_tune_set(op, api.conv_desc(*d), *WIDE, 1)


@pytest.mark.parametrize("variant,fits,others", [
    (NARROW, (64, 56, 56, 64, 64, 3, 3, 1, 1), [(16, 112, 112, 64, 64, 3, 3, 1, 1), (64, 112, 112, 64, 64, 3, 3, 2, 1), (64, 58, 58, 64, 64, 3, 3, 1, 0)]),
    (WIDE, (16, 28, 28, 128, 128, 3, 3, 1, 1), [(1, 112, 112, 128, 128, 3, 3, 1, 1), (16, 30, 30, 128, 128, 3, 3, 1, 0)]),
])
def test_a_recorded_variant_is_for_layers_that_it_takes(variant, fits, others):
    """Layers of the same pixels, channels and taps share a recorded choice; those whose width, stride or padding the window kernel
    does not take have the plan that they have without it."""
    for op in (api.JZ_FWD, api.JZ_BWD_DATA):
        ones = [o for o in others if op == api.JZ_FWD or o[8] == fits[8] and o[7] == 1]     # backward-data: the pixels of the input count
        before = [plan(op, *o) for o in ones]
        try:
            api.jz_conv2d_tune_set(op, api.conv_desc(*fits), *variant, 1)
            assert ": window tile %dx%dx%d, %d wavefronts, ring %d" % variant in plan(op, *fits)
            for o, b in zip(ones, before):
                assert plan(op, *o).split(":")[0] == plan(op, *fits).split(":")[0], "another key"
                assert plan(op, *o) == b, o
        finally:
            api.jz_conv2d_tune_clear()


@pytest.mark.gpu
@pytest.mark.parametrize("variant,N,H,W,C,K,R", [
    (NARROW, 1, 4, 3, 64, 64, 3),        # 12 pixels: less than a fragment; the filter covers the image
    (NARROW, 3, 9, 63, 64, 72, 3),       # the widest image, 384 rows; a ragged second column of tiles
    (NARROW, 2, 16, 8, 64, 64, 3),       # exactly one tile
    (NARROW, 6, 7, 7, 64, 40, 5),        # 25 taps, six images in two tiles
    (WIDE, 1, 1, 7, 128, 128, 3),        # one row of pixels: two of three tap rows outside
    (WIDE, 2, 17, 63, 128, 136, 3),      # two windows, widest image
    (WIDE, 5, 7, 8, 192, 64, 3),         # three windows: the first is overwritten while the second is read
    (WIDE, 3, 11, 31, 256, 72, 5),       # 25 taps, widest image of that size, four windows
    (WIDE, 2, 15, 17, 64, 256, 3),       # one window of the kernel with two
])
def test_against_the_oracle(variant, N, H, W, C, K, R):
    import jzt
    case = inputs.conv_case((83,), N, H, W, C, K, R, R, 1, R // 2)
    with jzt.forced_variant(jzt.desc_of(case), *variant, ops=(api.JZ_FWD,)):
        jzt.conv_all_ops_full(case, ops=(0,))
    case = inputs.conv_case((84,), N, H, W, K // 8 * 8, C, R, R, 1, R // 2)     # backward-data reads the C channels of dy
    with jzt.forced_variant(jzt.desc_of(case), *variant, ops=(api.JZ_BWD_DATA,)):
        jzt.conv_all_ops_full(case, ops=(1,))


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [2, 3])
def test_split_by_windows(splits):
    import jzt
    case = inputs.conv_case((85,), 2, 13, 13, 320, 320, 3, 3, 1, 1)             # five windows: 3 + 2, 2 + 2 + 1
    with jzt.forced_variant(jzt.desc_of(case), *WIDE, splits=splits, ops=(api.JZ_FWD, api.JZ_BWD_DATA)):
        jzt.conv_all_ops_full(case, ops=(0, 1))


@pytest.mark.gpu
@pytest.mark.parametrize("variant,N,H,C", [(NARROW, 4, 24, 64), (WIDE, 5, 24, 192)])
def test_every_epilogue(variant, N, H, C):
    import test_gpu_conv_bn
    import test_gpu_conv_bn_bwd
    for residual in (False, True):
        test_gpu_conv_bn.run_case(api, N, H, C, 72, 3, 1, 1, key=1, variant=variant, residual=residual)
    test_gpu_conv_bn_bwd.run_case(api, N, H, 72, C, 3, 1, 1, key=1, variant=variant)
    for second in (False, True):
        test_gpu_conv_bn_bwd.run_block_end(api, N, H, 72, C, 3, 1, 1, key=3, variant=variant, second=second)


@pytest.mark.gpu
def test_zeros_outside_the_image_under_values_that_are_not_finite():
    """A tap outside the image contributes a zero of its own: rows next to it in memory, of another image, may hold anything."""
    N, H, C = 3, 8, 64
    x = torch.zeros(N, H, H, C, dtype=torch.float16, device="cuda")
    x[1] = float("inf")
    w = torch.ones(64, 3, 3, C, dtype=torch.float16, device="cuda") / 64
    y = torch.empty(N, H, H, 64, dtype=torch.float16, device="cuda")
    d = api.conv_desc(N, H, H, C, 64, 3, 3, 1, 1)
    import jzt
    with jzt.forced_variant(d, *NARROW, ops=(api.JZ_FWD,)):
        api.jz_conv2d_fwd(d, x, w, y, None)
    torch.cuda.synchronize()
    assert torch.all(y[0] == 0) and torch.all(y[2] == 0) and torch.all(torch.isposinf(y[1]))
