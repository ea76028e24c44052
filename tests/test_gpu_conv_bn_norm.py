"""A split reduction that also normalizes (splitk_reduce_norm: up to 256 rows, and rows x rows x splits up to 250000, from 129 rows on 150000) at
the edges of its passes, columns and split lanes; more takes the reduction and the normalization apart."""
import pytest

import test_gpu_conv_bn as fwd
import test_gpu_conv_bn_bwd as bwd
from test_gpu_conv_bn_split import jz  # noqa: F401

pytestmark = pytest.mark.gpu

# N, H, channels in, channels out, filter, pad, splits
EDGES = [
    (2, 2, 512, 16, 1, 0, 8),       # 8 rows, one workgroup
    (2, 8, 256, 40, 3, 1, 9),       # 128 rows: exactly one pass; 40 columns: half a workgroup's at the end
    (2, 8, 256, 40, 3, 1, 16),      # apart: more splits
    (129, 1, 1024, 24, 1, 0, 8),    # one row in the second pass
    (1, 16, 128, 1032, 3, 1, 2),    # 256 rows: the most, ragged columns
    (129, 1, 1024, 24, 1, 0, 16),   # apart: more splits
    (1, 16, 128, 1032, 3, 1, 3),
    (257, 1, 512, 64, 1, 0, 8),     # apart: more rows
]


@pytest.mark.parametrize("N,H,C,K,R,pad,splits", EDGES)
def test_reduce_and_normalize(jz, N, H, C, K, R, pad, splits):  # noqa: F811
    v = (64, 64, 64, 4, 4)
    fwd.run_case(jz, N, H, C, K, R, 1, pad, key=21, variant=v, splits=splits)
    fwd.run_case(jz, N, H, C, K, R, 1, pad, key=22, variant=v, splits=splits, residual=True)
    bwd.run_case(jz, N, H, K, C, R, 1, pad, key=23, variant=v, splits=splits)
    bwd.run_block_end(jz, N, H, K, C, R, 1, pad, key=23, variant=v, splits=splits)
    bwd.run_block_end(jz, N, H, K, C, R, 1, pad, key=24, variant=v, splits=splits, second=False)
