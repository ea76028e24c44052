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
