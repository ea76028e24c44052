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
    assert need > 16
    for room in (0, need - 16):
        assert jz.lib().jz_conv2d_bwd_weight_f32(ctypes.byref(d), A, A + (1 << 28), A + (1 << 29), A + (1 << 30) if room else None, room,
                                                 None) == jz.JZ_ERR_WORKSPACE


def call_f16(jz, op, d, a, b, out_shape, room):  # noqa: F811
    import jzt
    out = torch.full(out_shape, float("nan"), dtype=torch.float16, device="cuda")
    jz.bind_conv2d(op, d, jzt.to_dev(a), jzt.to_dev(b), out, torch.empty(room, dtype=torch.uint8, device="cuda") if room else None)()
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("part", [0.0, 0.5, 0.99])
def test_half_precision(jz, part):  # noqa: F811
    import jzt
    for cfg, ops in ((FEW_TILES, (jz.JZ_FWD, jz.JZ_BWD_DATA)), (WIDE_FILTER, (jz.JZ_BWD_WEIGHT,))):
        N, H, C, K, R = cfg
        od, x, w, dy = operands(*cfg, np.float16)
        d = jz.conv_desc(N, H, H, C, K, R, R, 1, R // 2)
        for op, a, b, shape, fn in ((jz.JZ_FWD, x, w, (N, H, H, K), oracle.conv_fwd), (jz.JZ_BWD_DATA, dy, w, (N, H, H, C), oracle.conv_bwd_data),
                                    (jz.JZ_BWD_WEIGHT, x, dy, (K, R, R, C), oracle.conv_bwd_weight)):
            if op in ops:
                need = jz.jz_conv2d_workspace_bytes(op, d)
                assert need > 0, "the case has to split"
                jzt.check_half_output(call_f16(jz, op, d, a, b, shape, int(part * need) & ~15), fn(od, a, b), 1e-3, "op %d" % op)


def test_strided_backward_data_without_a_workspace(jz):  # noqa: F811
    import jzt
    od, d = oracle.conv_desc(2, 16, 15, 40, 24, 3, 3, (2, 2), (1, 1)), jz.conv_desc(2, 16, 15, 40, 24, 3, 3, 2, 1)
    rng = inputs.rng_for(94)
    w, dy = inputs.he_normal_f32(rng, (24, 3, 3, 40), 360).astype(np.float16), inputs.normal_f16(rng, (2, od.P, od.Q, 24))
    jzt.check_half_output(call_f16(jz, jz.JZ_BWD_DATA, d, dy, w, (2, 16, 15, 40), 0), oracle.conv_bwd_data(od, dy, w), 1e-3, "bwd_data")


def test_static_scratch_holds_fewer_splits_of_a_layer_that_wants_more(jz):  # noqa: F811
    """1360 -> 72 channels, 5 x 5, 54 x 54 pixels: the plan wants more than the array's 64 MiB.  FP64 products per tap on the GPU;
    one FP16 rounding of FP32 sums, 1e-3."""
    N, H, C, K, R = 4, 54, 1360, 72, 5
    d = jz.conv_desc(N, H, H, C, K, R, R, 1, 2)
    assert jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_WEIGHT, d) > jz.JZ_STATIC_SCRATCH_BYTES
    g = torch.Generator(device="cuda").manual_seed(1)
    x, dy = (torch.randn(N, H, H, c, generator=g, device="cuda").half() for c in (C, K))
    dw = torch.full((K, R, R, C), float("nan"), dtype=torch.float16, device="cuda")
    jz.jz_conv2d_bwd_weight_static(d, x, dy, dw)
    xp = torch.nn.functional.pad(x.double(), (0, 0, 2, 2, 2, 2))
    dy64 = dy.double().reshape(-1, K).t().contiguous()
    want = torch.stack([torch.stack([dy64 @ xp[:, r:r + H, s:s + H].reshape(-1, C) for s in range(R)], 1) for r in range(R)], 1)
    err = ((dw.double() - want).norm() / want.norm()).item()
    assert err < 1e-3, err
