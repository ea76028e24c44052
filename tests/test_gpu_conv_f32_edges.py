"""GPU parity of the single-precision operations at the edges of the LDS-direct kernel: k tiles that straddle filter taps, one
residue of the stride at a time, scattered outputs, more than 32 taps, channels rounded up on copies, reductions that end
inside a tile, images smaller than a step of the pixel counters."""
import pytest

from test_gpu_conv_f32 import all_ops, jz  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [
    # N, H, W, C, K, R, S, stride, pad
    (1, 3, 2, 4, 4, 3, 2, (1, 1), (1, 1)),          # images of 6 pixels: several images per 16-pixel step
    (3, 5, 7, 16, 68, 3, 3, (1, 1), (1, 1)),        # whole taps per tile; 105 pixels (a tail of 9), 68 = one tile and 4
    (2, 9, 9, 20, 132, 3, 3, (1, 1), (1, 1)),       # taps straddle tiles
    (2, 13, 11, 32, 64, 4, 4, (2, 2), (1, 1)),      # four residues of four taps
    (1, 14, 14, 48, 80, 3, 3, (2, 2), (1, 1)),      # residues of 1, 2, 2 and 4 taps
    (2, 11, 10, 12, 40, 5, 5, (3, 2), (2, 1)),      # six residues: two launches; taps straddle tiles
    (3, 9, 9, 64, 36, 1, 1, (2, 2), (0, 0)),        # scattered rows and zeros between them
    (1, 12, 12, 16, 32, 7, 7, (1, 1), (3, 3)),      # 49 taps
    (2, 12, 9, 16, 24, 2, 2, (3, 3), (0, 0)),       # a filter smaller than its stride: the register-staged kernel
    (2, 8, 9, 3, 21, 5, 5, (2, 2), (2, 2)),         # three channels on copies of four
    (2, 7, 7, 30, 33, 3, 3, (1, 1), (1, 1)),
    (130, 1, 1, 129, 65, 1, 1, (1, 1), (0, 0)),
]


@pytest.mark.parametrize("cfg", EDGES, ids=lambda c: "x".join(str(v) for v in c).replace(" ", ""))
def test_edges(jz, cfg):  # noqa: F811
    N, H, W, C, K, R, S, st, pad = cfg
    all_ops(jz, N, H, W, C, K, R, S, st, pad, 5)
