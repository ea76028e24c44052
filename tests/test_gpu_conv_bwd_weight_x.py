"""Weight gradients whose x is read as a matrix, at a constant distance per tap, or by its pixels' offsets: images smaller than a
tile of the reduction, one row or one column, filters larger than the image, and layers on either side of the choice."""
import pytest

import jzt
from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, C, K, R, S, stride, pad
    (40, 2, 2, 16, 32, 3, 3, 1, 1),       # sixteen images in a tile of 64 pixels
    (70, 1, 1, 8, 24, 3, 3, 1, 1),        # an image of one pixel: only the middle tap meets it
    (9, 1, 37, 24, 40, 3, 3, 1, 1),       # one row
    (9, 41, 1, 24, 40, 3, 3, 1, 1),       # one column
    (3, 9, 7, 64, 72, 5, 5, 1, 2),        # ragged columns
    (2, 3, 3, 16, 16, 7, 7, 1, 3),        # a filter larger than the image
    (5, 13, 11, 48, 64, 3, 3, 1, 0),      # unit stride, output grid smaller than the input's
    (5, 13, 11, 48, 64, 3, 3, 1, 2),      # ... and larger
    (4, 15, 14, 32, 136, 3, 3, 2, 1),     # strided
    (6, 10, 9, 40, 72, 1, 1, 1, 0),       # a matrix
    (6, 10, 9, 40, 72, 1, 1, 2, 0),       # a strided one
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_weight_gradient(cfg):
    N, H, W, C, K, R, S, st, pad = cfg
    res = jzt.conv_all_ops_full(inputs.conv_case((7, CASES.index(cfg)), N, H, W, C, K, R, S, st, pad, loss_scale=8.0), ops=(2,))
    print(res)
