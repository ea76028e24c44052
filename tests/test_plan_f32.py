"""Plans of the single-precision operations (host logic only)."""
import pytest

from test_gpu_conv_f32_window import FORMS, SHAPES, window_form
from test_plan_splits import jz  # noqa: F401


def test_the_layers_of_the_window_tests_run_on_that_kernel(jz):  # noqa: F811
    for cfg, forms in zip(SHAPES, FORMS):
        assert tuple(window_form(jz, op, cfg) for op in (jz.JZ_FWD, jz.JZ_BWD_DATA)) == forms, cfg
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        assert {f[op][:2] for f in FORMS if f[op]} == {(64, 192), (64, 256), (128, 192), (128, 256)}      # every variant


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
