"""Single-precision 3x3 layers whose output grid is their input grid: a tile's pixels taken apart once for all nine taps.  The sizes are
such that the plan takes that kernel, which the tests look up: the widest image that fits the window and both window lengths, narrow and
single-row images, ragged pixels and columns, both tile widths, whole and split reductions.  test_plan_f32.py asks the plans on the CPU."""
import re

import numpy as np
import pytest

from test_gpu_conv_f32 import check_f32, jz, run_f32  # noqa: F401  (jz is a fixture)
from test_gpu_conv_f32_parts import calls, operands

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, H, W, C, K, R, S, stride, pad
    (12, 43, 63, 64, 64, 3, 3, 1, 1),     # the widest image, 64-wide tiles
    (32, 33, 31, 96, 64, 3, 3, 1, 1),     # the widest of the short window
    (26, 39, 32, 64, 56, 3, 3, 1, 1),     # the narrowest of the long one, ragged columns (backward: not this kernel)
    (728, 9, 5, 64, 64, 3, 3, 1, 1),      # several images under a tile
    (818, 1, 40, 64, 64, 3, 3, 1, 1),     # one row: two thirds of the taps lie outside
    (818, 40, 1, 64, 64, 3, 3, 1, 1),     # one column
    (14, 61, 37, 32, 64, 3, 3, 1, 1),     # forward not this kernel; backward two pairs of windows
    (43, 28, 28, 128, 128, 3, 3, 1, 1),   # the last rows of tiles split
    (60, 14, 14, 256, 256, 3, 3, 1, 1),
    (12, 43, 63, 64, 128, 3, 3, 1, 1),    # 128-wide tiles forward, both window lengths
    (32, 33, 31, 64, 128, 3, 3, 1, 1),
    (24, 43, 63, 128, 64, 3, 3, 1, 1),    # and backward
    (64, 33, 31, 128, 64, 3, 3, 1, 1),
    (40, 56, 22, 32, 96, 3, 3, 1, 1),     # the shortest reduction forward: one pair of windows
    (15, 57, 11, 192, 96, 3, 3, 1, 1),    # 128-wide tiles, every row of tiles split
    (27, 11, 44, 96, 256, 3, 3, 1, 1),
    (49, 1, 45, 416, 32, 3, 3, 1, 1),     # a long reduction in many splits
    (18, 22, 22, 128, 64, 3, 3, 1, 1),    # backward whole where the plan without a window has three splits
    (30, 16, 16, 384, 448, 3, 3, 1, 1),   # backward, 252 k tiles: runs of 18
    (26, 39, 32, 64, 62, 3, 3, 1, 1),     # results written one by one; backward on copies with 64 channels
    (26, 39, 32, 62, 64, 3, 3, 1, 1),     # the other way round
]
# columns of a tile, rows of its window and the rows of tiles whose reduction is split, forward and backward-data; None: another kernel
FORMS = [
    ((64, 256, "none"), (64, 256, "none")),
    ((64, 192, "none"), (64, 192, "none")),
    ((64, 256, "none"), None),
    ((64, 192, "none"), (64, 192, "none")),
    ((64, 256, "none"), (64, 256, "none")),
    ((64, 192, "none"), (64, 192, "none")),
    (None, (64, 256, "none")),
    ((64, 192, "last"), (64, 192, "last")),
    ((64, 192, "last"), (64, 192, "last")),
    ((128, 256, "none"), (64, 256, "none")),
    ((128, 192, "none"), (64, 192, "none")),
    ((64, 256, "none"), (128, 256, "none")),
    ((64, 192, "none"), (128, 192, "none")),
    ((128, 192, "none"), (64, 192, "none")),
    ((128, 192, "all"), (64, 192, "none")),
    ((64, 256, "none"), (128, 256, "all")),
    ((64, 256, "all"), None),
    (None, (64, 192, "none")),
    ((64, 192, "none"), (64, 192, "last")),
    ((64, 256, "none"), (64, 256, "none")),
    ((64, 256, "none"), (64, 256, "none")),
]


def window_form(jz, op, cfg):  # noqa: F811
    """what FORMS has, as the library plans it"""
    m = re.search(r"window of (\d+) rows, rounded \d+ times \(\d+ without\), tile 128x(\d+), \d+ x \d+ tiles, (\d+) splits of \d+ k tiles, (\d+) rows",
                  jz.jz_conv2d_f32_describe_plan(op, jz.conv_desc(*cfg)))
    if not m:
        return None
    rows, bn, splits, full = (int(v) for v in m.groups())
    return bn, rows, "none" if splits == 1 else "last" if full else "all"


@pytest.mark.parametrize("cfg", SHAPES, ids=str)
def test_accuracy(jz, cfg):  # noqa: F811
    od, x, w, dy = operands(cfg, 200 + SHAPES.index(cfg))
    d = jz.conv_desc(*cfg)
    ops = calls(jz, od, x, w, dy)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        assert window_form(jz, op, cfg) == FORMS[SHAPES.index(cfg)][op], op
        a, b, shape, fn, red = ops[op]
        err, _ = check_f32(run_f32(jz, op, d, a, b, shape), fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)
        # the bar of the kernel that takes every tap's values apart: the same products, the large sums rounded once in 16 steps
        assert err <= 2.0 ** -24 * (2 + 2 * (red / 16) ** 0.5), (op, err)
        if FORMS[SHAPES.index(cfg)][op]:
            # A sum of n terms is off by n / 2 roundings of its final size, those of the plan's sums and of sums of sums together by
            # half their number; joining the small sums and what is left out of the products count as two more.  A rounding is
            # evenly spread over +- 2^-24: 2^-24 / sqrt(3) in the mean square.
            times = int(re.search(r"rounded (\d+) times", jz.jz_conv2d_f32_describe_plan(op, d))[1])
            assert err <= 2.0 ** -24 * ((times / 2 + 1) / 3) ** 0.5, (op, err, times)


@pytest.mark.parametrize("cfg", [SHAPES[1], SHAPES[7], SHAPES[8], SHAPES[9], SHAPES[11], SHAPES[14], SHAPES[15]], ids=str)
def test_values_that_parts_cannot_hold(jz, cfg):  # noqa: F811
    """A tile with such a value is computed again with the FP32 instructions, its share of a split reduction too: in the window
    kernel's order, channels outside and taps inside."""
    for value in (3.4e38, np.inf, np.nan):
        od, x, w, dy = operands(cfg, 230, (1.0, 0.01))
        x[0, 3, 2, 7] = x[-1, -1, -1, -1] = value
        dy[0, 2, 4, 9] = dy[-1, 0, 0, -1] = value
        d = jz.conv_desc(*cfg)
        ops = calls(jz, od, x, w, dy)
        for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
            a, b, shape, fn, red = ops[op]
            got = run_f32(jz, op, d, a, b, shape)
            ref, mag = fn(od, a, b), fn(od, np.abs(a), np.abs(b))
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref)), op
            ok = np.isfinite(ref)
            check_f32(got[ok], ref[ok], mag[ok], "op %d" % op)


@pytest.mark.parametrize("part", [0.0, 0.5, 0.99])
@pytest.mark.parametrize("cfg", [SHAPES[7], SHAPES[8], SHAPES[16]], ids=str)
def test_less_workspace_than_reported(jz, cfg, part):  # noqa: F811
    """Fewer splits or none: the plan for the room there is, on this kernel or another."""
    from test_gpu_small_workspace import call_f32
    od, x, w, dy = operands(cfg, 240)
    d = jz.conv_desc(*cfg)
    ops = calls(jz, od, x, w, dy)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        a, b, shape, fn, _ = ops[op]
        need = jz.jz_conv2d_f32_workspace_bytes(op, d)
        if FORMS[SHAPES.index(cfg)][op]:
            assert need > 0, "the case has to split"
            check_f32(call_f32(jz, op, d, a, b, shape, int(part * need) & ~15), fn(od, a, b), fn(od, np.abs(a), np.abs(b)), "op %d" % op)
