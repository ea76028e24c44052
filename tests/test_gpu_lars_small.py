"""GPU parity of the LARS update where its launch scheme changes: the one-workgroup launch of small sets (at most four chunks
of 4096 elements, at most 64 tensors) and the two sizes of the per-tensor reduction."""
import numpy as np
import pytest
import torch

from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [1], [16384], [16385], [4096, 5, 4096, 8], [4097, 4097], [4097, 4097, 3],      # four chunks and five
    [0] * 61 + [5, 7, 4096], [0] * 62 + [5, 7, 4096],                              # 64 tensors and 65
    [10485760, 9], [10485761],                                                     # 2560 chunks and 2561 in one tensor
], ids=lambda s: "%dx%d" % (len(s), sum(s)))
@pytest.mark.parametrize("bad", [False, True])
def test_two_steps_against_the_oracle(sizes, bad):
    import jzt
    assert torch.cuda.is_available()
    ps = inputs.random_param_set((0, 77, len(sizes), sum(sizes) % 1000), sizes, loss_scale=256.0, momentum_std=1e-3,
                                 flags=[(3, 2, 1, 0)[i % 4] for i in range(len(sizes))])
    if bad:
        ps.grad16[-1] = np.float16(np.nan)
    r = jzt.LarsRun(ps)
    for _ in range(2):       # the second step takes the sums of squares of the weights that the first one left
        got = r.step()
        jzt.check_lars_against_oracle(ps, got)
        ps.master_w, ps.momentum, ps.weight16 = got[0].copy(), got[1].copy(), got[2].copy()
