"""The padded 4-channel copy of small-channel inputs: images of less than one and of several workgroups of the copy, tensors
that end inside a 16-byte chunk, every channel count, filter columns that make the padded rows wider than the image."""
import numpy as np
import pytest

from paper_1807_11205_amd import inputs
from test_gpu_conv import jz  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,C,K,R,S,pad", [(1, 5, 7, 3, 16, 3, 3, 1), (3, 33, 61, 1, 16, 3, 5, 2), (2, 47, 91, 3, 64, 7, 7, 3),
                                               (2, 64, 66, 4, 24, 5, 5, 0), (1, 90, 49, 2, 16, 3, 11, 2), (3, 3, 900, 3, 16, 3, 3, 1)])
def test_padded_copy_edges_against_the_oracle(jz, N, H, W, C, K, R, S, pad):  # noqa: F811
    import jzt
    import oracle
    od = oracle.conv_desc(N, H, W, C, K, R, S, 2, (pad, pad))
    d = jz.conv_desc(N, H, W, C, K, R, S, 2, (pad, pad))
    assert "4-channel padded copy" in jz.jz_conv2d_describe_plan(jz.JZ_BWD_WEIGHT, d)
    rng = inputs.rng_for(47, H, W, C)
    x = inputs.normal_f16(rng, (N, H, W, C))
    w = inputs.he_normal_f32(rng, (K, R, S, C), R * S * C).astype(np.float16)
    dy = inputs.normal_f16(rng, (N, od.P, od.Q, K), std=8.0)
    jzt.all_ops_against_the_oracle(d, od, x, w, dy, ops=(jz.JZ_FWD, jz.JZ_BWD_WEIGHT))
