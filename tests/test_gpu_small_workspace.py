"""Layers given less workspace than the plan asks for: forward and backward-data run with fewer splits, or none; a weight
gradient runs while what fits still fills the chip, and is refused otherwise.  Same bars as with the full workspace."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1807_11205_amd import inputs
from test_gpu_conv_f32 import check_f32, jz  # noqa: F401

pytestmark = pytest.mark.gpu

# N, H, C, K, R: a few tiles and a long reduction (forward / backward-data split), and a filter of more than 256 tiles
FEW_TILES = (4, 7, 192, 320, 3)
WIDE_FILTER = (16, 14, 640, 2048, 1)     # 320 tiles of 64 x 64, 3136 pixels


def operands(N, H, C, K, R, dtype):
    od = oracle.conv_desc(N, H, H, C, K, R, R, (1, 1), (R // 2, R // 2))
    rng = inputs.rng_for(93, N, H, C, K)
    x = rng.standard_normal((N, H, H, C), dtype=np.float32).astype(dtype)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32((2.0 / (R * R * C)) ** 0.5)).astype(dtype)
    dy = rng.standard_normal((N, H, H, K), dtype=np.float32).astype(dtype)
    return od, x, w, dy


def call_f32(jz, op, d, a, b, out_shape, room):  # noqa: F811
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    out = torch.full(out_shape, float("nan"), device="cuda")
    ws = torch.empty(room, dtype=torch.uint8, device="cuda") if room else None
    jz.jz_conv2d_f32(op, d, ta, tb, out, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("part", [0.0, 0.5, 0.99])
def test_single_precision(jz, part):  # noqa: F811
    N, H, C, K, R = FEW_TILES
    od, x, w, dy = operands(*FEW_TILES, np.float32)
    d = jz.conv_desc(N, H, H, C, K, R, R, 1, R // 2)
    for op, a, b, shape, fn in ((jz.JZ_FWD, x, w, (N, H, H, K), oracle.conv_fwd), (jz.JZ_BWD_DATA, dy, w, (N, H, H, C), oracle.conv_bwd_data)):
        need = jz.jz_conv2d_f32_workspace_bytes(op, d)
        assert need > 0, "the case has to split"
        got = call_f32(jz, op, d, a, b, shape, int(part * need) & ~15)
        check_f32(got, fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)
    N, H, C, K, R = WIDE_FILTER
    od, x, w, dy = operands(*WIDE_FILTER, np.float32)
    d = jz.conv_desc(N, H, H, C, K, R, R, 1, R // 2)
    need = jz.jz_conv2d_f32_workspace_bytes(jz.JZ_BWD_WEIGHT, d)
    assert need > 0, "the case has to split"
    got = call_f32(jz, jz.JZ_BWD_WEIGHT, d, x, dy, (K, R, R, C), int(part * need) & ~15)
    check_f32(got, oracle.conv_bwd_weight(od, x, dy), oracle.conv_bwd_weight(od, np.abs(x), np.abs(dy)), "weight gradient")


def test_single_precision_weight_gradient_that_would_leave_the_chip_idle_is_refused(jz):  # noqa: F811
    d = jz.conv_desc(16, 20, 20, 8, 8, 3, 3, 1, 1)         # one tile
    need = jz.jz_conv2d_f32_workspace_bytes(jz.JZ_BWD_WEIGHT, d)
    A = 0x10000000                                         # refused before anything is launched
    for room in (0, need - 16):
        assert jz.lib().jz_conv2d_bwd_weight_f32(ctypes.byref(d), A, A + (1 << 28), A + (1 << 29), A + (1 << 30) if room else None, room,
                                                 None) == jz.JZ_ERR_WORKSPACE
