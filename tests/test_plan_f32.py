"""Plans of the single-precision operations (host logic only)."""
import random
import re

import pytest

from test_gpu_conv_f32_window import FORMS, SHAPES, window_form
from test_plan_splits import jz  # noqa: F401


def test_the_layers_of_the_window_tests_run_on_that_kernel(jz):  # noqa: F811
    for cfg, forms in zip(SHAPES, FORMS):
        assert tuple(window_form(jz, op, cfg) for op in (jz.JZ_FWD, jz.JZ_BWD_DATA)) == forms, cfg
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        assert {f[op][:2] for f in FORMS if f[op]} == {(64, 192), (64, 256), (128, 192), (128, 256)}      # every variant


def roundings(tile_n, k_tiles, parts):
    """How often a large sum of the window kernel is rounded: 64-wide tiles start a new one every nine or 18 k tiles."""
    if tile_n == 128:
        return k_tiles + (parts if parts > 1 else 0)
    return min(run + (k_tiles // run if run < k_tiles else 0) for run in (9, 18)) + (parts if parts > 1 else 0)


def test_no_sum_is_rounded_more_often_with_a_window_than_without(jz):  # noqa: F811
    """18x22x22 and the like, 64 output channels backward, ran in 20 roundings where three splits of 12 k tiles have 15."""
    rng = random.Random(5)
    layers = [(18, 22, 22, 128, 64), (9, 34, 34, 128, 64), (4, 49, 49, 128, 64), (2, 57, 57, 160, 64), (6, 18, 18, 640, 64), (64, 56, 56, 64, 64),
              (64, 28, 28, 128, 128), (64, 14, 14, 256, 256), (57, 24, 24, 448, 288)]
    layers += [(rng.choice((1, 4, 18, 64)), rng.randint(1, 63), rng.randint(1, 63), 32 * rng.randint(1, 16), 32 * rng.randint(1, 16)) for _ in range(3000)]
    seen = 0
    for N, H, W, C, K in layers:
        for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
            text = jz.jz_conv2d_f32_describe_plan(op, jz.conv_desc(N, H, W, C, K, 3, 3, 1, 1))
            m = re.search(r"rounded (\d+) times \((\d+) without\), tile 128x(\d+), .* (\d+) splits of (\d+) k tiles, (\d+) rows", text)
            if not m:
                continue
            here, without, tile_n, splits, per_split, whole_rows = (int(v) for v in m.groups())
            want = roundings(tile_n, per_split, splits)
            if whole_rows:
                want = max(want, roundings(tile_n, 9 * (C if op == jz.JZ_FWD else K) // 16, 1)) if splits > 1 else want
            assert want == here <= without, (N, H, W, C, K, op, text)
            seen += 1
    assert seen > 2000


def test_128_wide_tiles_with_a_window_are_not_split_into_parts_of_18_k_tiles(jz):  # noqa: F811
    """4 to 12 % slower than the plan without a window; 64-wide tiles gain with such parts."""
    rng = random.Random(6)
    layers = [((30, 33, 11, 160, 96), 0), ((8, 36, 38, 96, 160), 1), ((21, 6, 56, 288, 96), 0)]
    layers += [((rng.randint(1, 40), rng.randint(1, 63), rng.randint(1, 63), 32 * rng.randint(1, 16), 32 * rng.randint(1, 16)), i % 2) for i in range(6000)]
    for cfg, op in layers:
        text = jz.jz_conv2d_f32_describe_plan(op, jz.conv_desc(*cfg, 3, 3, 1, 1))
        assert not re.search(r"window .* tile 128x128, .* ([2-9]|[1-9]\d+) splits of 18 k tiles", text), (cfg, text)


def test_no_window_reaches_past_32_bits(jz):  # noqa: F811
    """Rows behind the tensor, up to 128 and a row of the image, are requested: their offsets have to stay out of the tensor's range."""
    for N, H, W, C, K in ((3, 35, 3, 3047776, 28), (4, 36, 2, 3133216, 28), (1, 12, 13, 4062528, 8)):
        assert "window" not in jz.jz_conv2d_f32_describe_plan(jz.JZ_FWD, jz.conv_desc(N, H, W, C, K, 3, 3, 1, 1))
        assert "window" not in jz.jz_conv2d_f32_describe_plan(jz.JZ_BWD_DATA, jz.conv_desc(N, H, W, K, C, 3, 3, 1, 1))


@pytest.mark.parametrize("cfg, op, words", [
    ((64, 7, 7, 512, 512, 3, 3, 1, 1), 2, ("M 512 N 4608 K 3136", "parts", "splits")),
    ((4, 9, 9, 64, 64, 3, 3, 2, 1), 1, ("residues of the stride",)),
    ((2, 8, 8, 20, 16, 3, 3, 1, 1), 0, ("per-lane taps",)),
    ((8, 32, 32, 3, 64, 7, 7, 2, 3), 0, ("K 196", "copies of 4 n channels")),
    ((2, 8, 8, 1, 16, 3, 3, 1, 1), 0, ("operands through registers",)),
])
def test_a_plan_says_what_runs(jz, cfg, op, words):  # noqa: F811
    text = jz.jz_conv2d_f32_describe_plan(op, jz.conv_desc(*cfg))
    assert all(w in text for w in words) and "window" not in text, text
