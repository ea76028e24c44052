"""Statistics left by a split reduction (splitk_reduce_stats) at the edges of its slabs, columns and split lanes: the
convolution's result keeps the bits of the plain call, the normalization built on the sums meets the oracle."""
import pytest
import torch

import test_gpu_conv_bn as fwd
import test_gpu_conv_bn_bwd as bwd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    assert torch.cuda.is_available()
    return api


# N, H, channels in, channels out, filter, pad, splits
EDGES = [
    (1, 3, 512, 72, 3, 1, 24),      # 9 rows: less than one pass; 72 columns: a ragged column group
    (1, 4, 256, 2048, 3, 1, 9),     # 16 rows: exactly one pass
    (2, 5, 1024, 64, 1, 0, 16),     # 50 rows, one column group, a split per slice
    (17, 8, 128, 136, 3, 1, 2),     # 1088 rows: two slabs' worth of passes at 64 slabs
    (64, 14, 64, 64, 3, 1, 5),      # 12544 rows: more than 64 slabs, finished by the finalize launch
]


@pytest.mark.parametrize("N,H,C,K,R,pad,splits", EDGES)
def test_split_reduction_statistics(jz, N, H, C, K, R, pad, splits):
    v = (64, 64, 64, 4, 4)
    fwd.run_case(jz, N, H, C, K, R, 1, pad, key=11, variant=v, splits=splits)
    fwd.run_case(jz, N, H, C, K, R, 1, pad, key=12, variant=v, splits=splits, residual=True)
    # the backward-data product of the layer with the channel counts exchanged has the same matrix sizes
    bwd.run_case(jz, N, H, K, C, R, 1, pad, key=13, variant=v, splits=splits)
    bwd.run_block_end(jz, N, H, K, C, R, 1, pad, key=13, variant=v, splits=splits)
    bwd.run_block_end(jz, N, H, K, C, R, 1, pad, key=14, variant=v, splits=splits, second=False)
