"""GPU parity of batch normalization around the number of partial sums up to which the apply pass adds them up itself: the last
tensor that does and the first that does not, channel counts that are not multiples of its 64, rows that end inside a pass."""
import pytest

from test_gpu_bn import _inputs, _run, jz  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,C", [(4096, 256), (4097, 256), (4160, 256), (2049, 72), (33, 2040), (127, 8), (64 * 128 + 1, 128)])
@pytest.mark.parametrize("relu", [True, False])
def test_merged_apply_passes(jz, rows, C, relu):  # noqa: F811
    _run(jz, *_inputs((rows, C, 7), rows, C), 1e-5, relu)
