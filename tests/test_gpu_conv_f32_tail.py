"""Single-precision layers whose last, unfilled round of workgroups alone splits the reduction: rows computed whole and rows
put together from partial sums meet inside one result, at ragged last tiles both ways."""
import pytest

from test_gpu_conv_f32 import all_ops, jz  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, C, K, R: forward or backward-data splits its tail
    (7, 28, 512, 132, 1),       # forward: the last tile rows, 132 columns (a ragged column of tiles)
    (21, 13, 260, 512, 1),      # backward-data, 3549 rows (a ragged last row of tiles)
    (17, 14, 64, 260, 3),       # forward with padding taps in the tail
    (13, 14, 512, 512, 1),      # most of the rows are tail
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_split_tail(jz, cfg):  # noqa: F811
    N, H, C, K, R = cfg
    d = jz.conv_desc(N, H, H, C, K, R, R, 1, R // 2)
    ws = [jz.jz_conv2d_f32_workspace_bytes(op, d) for op in (jz.JZ_FWD, jz.JZ_BWD_DATA)]
    whole = [N * H * H * K * 4, N * H * H * C * 4]
    assert any(0 < w < m for w, m in zip(ws, whole)), "neither operation has partial sums for a part of its rows"
    all_ops(jz, N, H, H, C, K, R, R, (1, 1), (R // 2, R // 2), 6)
