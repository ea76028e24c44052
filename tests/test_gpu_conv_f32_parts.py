"""Single-precision layers whose operands are taken apart into three bfloat16 values: accuracy of FP32 at the edges of tiles and
reductions, and values that the parts cannot hold."""
import numpy as np
import pytest
import torch

import oracle
from paper_1807_11205_amd import inputs
from test_gpu_conv_f32 import check_f32, jz, run_f32  # noqa: F401  (jz is a fixture)

pytestmark = pytest.mark.gpu


def operands(cfg, key, scale=(1.0, 1.0)):
    N, H, W, C, K, R, S, st, pad = cfg
    od = oracle.conv_desc(N, H, W, C, K, R, S, st, (pad, pad))
    rng = inputs.rng_for(94, key, N, H, C, K, R)
    x = rng.standard_normal((N, H, W, C), dtype=np.float32) * np.float32(scale[0])
    w = rng.standard_normal((K, R, S, C), dtype=np.float32) * np.float32((2.0 / (R * S * C)) ** 0.5 * scale[1])
    dy = rng.standard_normal((N, od.P, od.Q, K), dtype=np.float32) * np.float32(scale[0])
    return od, x, w, dy


def calls(jz, od, x, w, dy):
    """op: (first and second input, output shape, oracle, length of the reduction)"""
    return {jz.JZ_FWD: (x, w, dy.shape, oracle.conv_fwd, w[0].size), jz.JZ_BWD_DATA: (dy, w, x.shape, oracle.conv_bwd_data, w[..., 0].size),
            jz.JZ_BWD_WEIGHT: (x, dy, w.shape, oracle.conv_bwd_weight, dy[..., 0].size)}


SHAPES = [
    # N, H, W, C, K, R, S, stride, pad
    (8, 28, 28, 64, 64, 3, 3, 1, 1),      # whole tiles, split reductions
    (9, 20, 20, 20, 64, 5, 5, 1, 2),      # a reduction of 500: flattened taps, an odd number of k tiles, a partial one
    (6, 28, 28, 48, 136, 3, 3, 1, 1),     # ragged columns
    (12, 28, 28, 32, 192, 1, 1, 1, 0),    # two k tiles: nothing left to request behind the first
    (33, 14, 14, 64, 48, 1, 1, 1, 0),     # three k tiles backwards
    (7, 27, 29, 64, 128, 3, 3, 2, 1),     # residues of a stride: one, two and four taps
    (40, 14, 14, 128, 256, 1, 1, 2, 0),   # scattered results
    (2, 56, 56, 64, 64, 7, 7, 1, 3),      # more than 32 taps
    (24, 28, 28, 128, 128, 3, 3, 1, 1),   # 128-wide tiles
    (64, 1, 1, 2048, 1000, 1, 1, 1, 0),   # a fully connected layer: four k tiles in the weight gradient
]


@pytest.mark.parametrize("cfg", SHAPES)
def test_accuracy(jz, cfg):
    od, x, w, dy = operands(cfg, SHAPES.index(cfg))
    d = jz.conv_desc(*cfg)
    for op, (a, b, shape, fn, red) in calls(jz, od, x, w, dy).items():
        err, _ = check_f32(run_f32(jz, op, d, a, b, shape), fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)
        # what is left out of a product is at most 2^-24 of it, of either sign: 2^-24 of the result.  The large sums are rounded once
        # in 16 steps, each time by at most 2^-24 of the sum, which grows as sqrt(k): sqrt(k / 16) 2^-24.  Adding the small sums rounds
        # by half an ulp, the result by another: 2^-24 together.  The FP32 form, which short launches may take, rounds four times as
        # often: twice the second.
        assert err <= 2.0 ** -24 * (2 + 2 * (red / 16) ** 0.5), (op, err)


# the last four: sums that are too large for the loop once scaled, operands that are (some, all), and sums on either side of that
@pytest.mark.parametrize("scale", [(1e-20, 1e15), (1e25, 1e-20), (1e-30, 1.0), (1e18, 1e18), (2.0 ** 104, 1e-20), (1e-20, 2.0 ** 110), (2.0 ** 50, 2.0 ** 22)])
def test_magnitudes(jz, scale):
    cfg = SHAPES[0]
    od, x, w, dy = operands(cfg, 50, scale)
    d = jz.conv_desc(*cfg)
    ops = calls(jz, od, x, w, dy)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        a, b, shape, fn, red = ops[op]
        check_f32(run_f32(jz, op, d, a, b, shape), fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)


# Operands whose third part, second part, and whole value would be too small for a bfloat16 (2^-126, subnormal down to 2^-133), the
# other operand such that results are ordinary numbers; the last two hold the values of a subnormal operand (eight bits and one).
@pytest.mark.parametrize("small", [2.0 ** -104, 2.0 ** -109, 2.0 ** -113, 1e-35, 2.0 ** -120, 1e-37, 2.0 ** -141, 2.0 ** -148])
@pytest.mark.parametrize("cfg", [SHAPES[0], SHAPES[5], (24, 28, 28, 128, 128, 3, 3, 1, 1)], ids=["64", "residues", "128"])
def test_small_operands_keep_their_bits(jz, cfg, small):
    other = min(1.0 / small, 1e30)
    for key, scale in ((70, (small, other)), (71, (other, small))):
        od, x, w, dy = operands(cfg, key, scale)
        d = jz.conv_desc(*cfg)
        ops = calls(jz, od, x, w, dy)
        for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
            a, b, shape, fn, red = ops[op]
            err, _ = check_f32(run_f32(jz, op, d, a, b, shape), fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)
            assert err <= 2.0 ** -24 * (2 + 2 * (red / 16) ** 0.5), (op, scale, err)  # as in test_accuracy


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, -3.4e38])
@pytest.mark.parametrize("cfg", [SHAPES[0], SHAPES[5], (24, 28, 28, 128, 128, 3, 3, 1, 1)], ids=["64", "residues", "128"])
def test_values_that_parts_cannot_hold(jz, cfg, value):
    """Infinities, NaN, and values that round to an infinite bfloat16 (the filters keep their products finite)."""
    od, x, w, dy = operands(cfg, 60, (1.0, 0.01))
    x[0, 3, 5, 7] = x[-1, -1, -1, -1] = value
    dy[0, 2, 4, 9] = value
    d = jz.conv_desc(*cfg)
    ops = calls(jz, od, x, w, dy)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA) if abs(value) < np.inf else (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT):
        a, b, shape, fn, red = ops[op]
        got = run_f32(jz, op, d, a, b, shape)
        ref, mag = fn(od, a, b), fn(od, np.abs(a), np.abs(b))
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref)), op
        assert np.array_equal(got[np.isinf(ref)] > 0, ref[np.isinf(ref)] > 0), op
        ok = np.isfinite(ref)
        check_f32(got[ok], ref[ok], mag[ok], "op %d" % op)
