"""Workspace demands (host logic only): what a split reduction asks for is bounded, and what needs no room asks for none."""
import pytest

from paper_1807_11205_amd import shapes

MB = 1 << 20


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    return api


# long reductions into wide results: without a bound the cost model would take 0.4 to 3 GB of partial sums
LONG = [(29, 102, 867, 1477, 5, 1), (60, 60, 1048, 1512, 5, 1), (37, 111, 2032, 800, 3, 2), (32, 128, 400, 1576, 7, 2),
        (13, 56, 1240, 552, 3, 1), (4, 100, 2048, 2048, 1, 1), (16, 64, 2048, 2048, 1, 1), (24, 46, 2048, 1024, 3, 1)]


def test_partial_sums_of_single_precision_layers_are_bounded(jz):
    for N, H, C, K, R, st in LONG:
        C, K = C // 4 * 4, K // 4 * 4        # no copies of operands: the demand is partial sums
        d = jz.conv_desc(N, H, H, C, K, R, R, st, R // 2)
        for op in (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT):
            assert jz.jz_conv2d_f32_workspace_bytes(op, d) <= 256 * MB, (N, H, C, K, R, st, op)
    for v in ("v1", "v1.5"):
        for N in (2, 7, 24, 64, 200):
            for c in shapes.resnet50_convs(v):
                if c.C % 4 == 0:
                    d = jz.conv_desc(N, c.H, c.H, c.C, c.K, c.R, c.R, c.stride, c.pad)
                    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT):
                        assert jz.jz_conv2d_f32_workspace_bytes(op, d) <= 256 * MB


def test_partial_sums_of_half_precision_layers_are_bounded(jz):
    for N, H, C, K, R, st in LONG:
        C, K = C // 8 * 8, K // 8 * 8
        d = jz.conv_desc(N, H, H, C, K, R, R, st, R // 2)
        for op in (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT):
            assert jz.jz_conv2d_workspace_bytes(op, d) <= 256 * MB, (N, H, C, K, R, st, op)


def test_strided_backward_data_of_ragged_channels_asks_for_no_workspace(jz):
    for N, H, W, C, K, R, S, st, pad in ((2, 16, 15, 40, 24, 3, 3, 2, 1), (1, 20, 20, 8, 200, 7, 4, (3, 2), (2, 1))):
        assert jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_DATA, jz.conv_desc(N, H, W, C, K, R, S, st, pad)) == 0


def whole_plan(rows, C):
    """Slabs of batch normalization in one launch: 64 channels a workgroup, at most 256 of them, and the fewest rows that pay for one more."""
    least = 256 if rows <= 256 or rows >= 4096 else 128
    return -(-rows // max(least, -(-rows // (256 // (C // 64)))))


def test_batch_normalization_in_one_launch_has_room_for_all_its_workgroups(jz):
    """Two FP64 sums a channel of every slab, and behind them a flag a workgroup or the coefficients of the launches apart."""
    for rows, C in ((1, 64), (63, 64), (64, 128), (257, 64), (2048, 64), (6272, 64), (16384, 64), (25088, 64), (49, 2048), (12545, 128), (4099, 1984),
                    (100352, 64), (200704, 64), (802816, 64)):
        slabs = whole_plan(rows, C)
        assert jz.jz_bn_workspace_bytes(rows, C) >= slabs * 2 * C * 8 + max(16 * C, slabs * C // 8), (rows, C)
    for N, H, C, K in ((1, 7, 64, 64), (1, 14, 64, 128), (2, 28, 128, 128), (64, 56, 64, 64)):
        d, rows = jz.conv_desc(N, H, H, C, K, 1, 1, 2, 0), N * H * H
        need = jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_DATA, d) + whole_plan(rows, C) * (2 * C * 8) + 16 * C
        assert jz.jz_conv2d_bwd_data_bn_relu_bwd_workspace_bytes(d) >= need, (N, H, C, K)
