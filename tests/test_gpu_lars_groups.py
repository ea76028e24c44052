"""GPU parity of the LARS update where a workgroup of its reduce pass takes a group of chunks of 4096 elements: the largest sets
of each group size and the first beyond, tensors that start between 16-byte boundaries, last chunks of every kind, the sets
with one very large tensor, and more tensors than groups.  A fresh workspace, carried sums of the weights, an overflow between."""
import numpy as np
import pytest
import torch

from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu
CH = 4096
SIZES = [
    [512 * CH], [512 * CH + 1], [511 * CH, 5, CH + 3],              # 512 chunks one by one, 513 and 514 in pairs
    [1024 * CH - 7, 8], [1200 * CH + 9, 16, 300 * CH + 4],          # groups of four chunks, ends inside a 16-byte piece
    [3, 700 * CH + 5, 90 * CH, 1],                                  # tensors that start between 16-byte boundaries
    [1536 * CH], [1536 * CH + 8],                                   # the last set that takes groups, the first that does not
    [2561 * CH + 12, 40], [8] * 512, [8] * 513, [2600 * CH] + [8] * 512,
]


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: "%dx%d" % (len(s), sum(s)))
def test_steps_with_an_overflow_between_them(sizes):
    import jzt
    assert torch.cuda.is_available()
    ps = inputs.random_param_set((0, 79, len(sizes), sum(sizes) % 1000), sizes, loss_scale=256.0, momentum_std=1e-3,
                                 flags=[(3, 2, 1, 0)[i % 4] for i in range(len(sizes))])
    good = ps.grad16.copy()
    r = jzt.LarsRun(ps)
    for step in range(3):
        ps.grad16[:] = good
        if step == 1:
            ps.grad16[-1] = np.float16(-np.inf)
        r.g.copy_(torch.from_numpy(ps.grad16))
        got = r.step()
        out = jzt.check_lars_against_oracle(ps, got)
        assert out["flag"] == (1 if step == 1 else 0)
        ps.master_w, ps.momentum, ps.weight16 = got[0].copy(), got[1].copy(), got[2].copy()
