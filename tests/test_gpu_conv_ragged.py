"""GPU parity of convolutions whose channel counts fill no k tile: the flattened (tap, channel) reduction (multiples of 8)
and the zero-extended copies (counts that are not multiples of 8), against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    assert torch.cuda.is_available()
    return api


RAGGED = [
    # N, H, W, C, K, R, S, stride, pad
    (1, 5, 7, 8, 8, 3, 3, 1, 1),          # the smallest: nine taps in 72 elements, several taps per 16-byte row of chunks
    (2, 14, 14, 16, 16, 3, 3, 1, 1),
    (3, 13, 11, 24, 136, 3, 3, 1, 1),     # one tile and a bit in n, taps straddle tiles
    (2, 9, 9, 200, 72, 5, 5, 1, 2),       # 25 taps, long reduction
    (2, 12, 10, 40, 56, 2, 3, 1, 0),      # no padding
    (2, 16, 15, 40, 24, 3, 3, 2, 1),      # strided: backward-data by residues of the stride
    (1, 20, 20, 8, 200, 7, 4, (3, 2), (2, 1)),
    (4, 17, 17, 48, 80, 4, 8, 1, (1, 3)),  # exactly 32 taps
    # counts that are not multiples of 8
    (2, 9, 8, 37, 50, 3, 3, 1, 1),
    (2, 9, 8, 64, 33, 3, 3, 2, 1),        # only the output channels
    (3, 7, 7, 100, 96, 1, 1, 1, 0),       # only the input channels
    (5, 4, 4, 130, 129, 1, 1, 2, 0),
    (64, 1, 1, 500, 999, 1, 1, 1, 0),     # a classifier
]


@pytest.mark.parametrize("cfg", RAGGED, ids=lambda c: "x".join(str(v) for v in c).replace(" ", ""))
def test_ragged_channels(jz, cfg):
    import jzt
    N, H, W, C, K, R, S, st, pad = cfg
    st, pad = ((v, v) if isinstance(v, int) else v for v in (st, pad))
    od, d = oracle.conv_desc(N, H, W, C, K, R, S, st, pad), jz.conv_desc(N, H, W, C, K, R, S, st, pad)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT):
        assert "element-wise" not in jz.jz_conv2d_describe_plan(op, d)
    rng = inputs.rng_for(31, N, H, C, K, R)
    x = inputs.normal_f16(rng, (N, H, W, C))
    w = inputs.he_normal_f32(rng, (K, R, S, C), R * S * C).astype(np.float16)
    dy = inputs.normal_f16(rng, (N, od.P, od.Q, K), std=8.0)
    jzt.all_ops_against_the_oracle(d, od, x, w, dy)


def test_without_room_for_the_copies_the_element_wise_kernel_runs(jz):
    import jzt
    N, H, C, K = 2, 9, 37, 50
    od, d = oracle.conv_desc(N, H, H, C, K, 3, 3, (1, 1), (1, 1)), jz.conv_desc(N, H, H, C, K, 3, 3, 1, 1)
    rng = inputs.rng_for(32)
    x, w = inputs.normal_f16(rng, (N, H, H, C)), inputs.he_normal_f32(rng, (K, 3, 3, C), 9 * C).astype(np.float16)
    y = torch.full((N, H, H, K), float("nan"), dtype=torch.float16, device="cuda:0")
    jz.jz_conv2d_fwd(d, jzt.to_dev(x), jzt.to_dev(w), y, None)
    jzt.check_half_output(y.cpu().numpy(), oracle.conv_fwd(od, x, w), 1e-3, "fwd")
