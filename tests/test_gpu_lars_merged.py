"""GPU parity of the LARS update of sets of 5 to 256 chunks of 4096 elements, whose update launch works out its own rates, and
of the first set beyond: a fresh workspace, carried sums of the weights, an overflow in between.  The loss scale on
the device (its controller runs in the same launch) is covered by the loss-scale tests, whose sets are of this size."""
import numpy as np
import pytest
import torch

from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [[16384, 1], [4097, 4097, 7, 9000], [1] * 255 + [4096], [1] * 256 + [5], [1044480, 4090], [1048576], [1048577]]


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: "%dx%d" % (len(s), sum(s)))
def test_steps_with_an_overflow_between_them(sizes):
    import jzt
    assert torch.cuda.is_available()
    ps = inputs.random_param_set((0, 78, len(sizes), sum(sizes) % 1000), sizes, loss_scale=256.0, momentum_std=1e-3,
                                 flags=[(3, 2, 1, 0)[i % 4] for i in range(len(sizes))])
    good = ps.grad16.copy()
    r = jzt.LarsRun(ps)
    for step in range(4):
        ps.grad16[:] = good
        if step == 2:
            ps.grad16[len(good) // 2] = np.float16(np.inf)
        r.g.copy_(torch.from_numpy(ps.grad16))
        got = r.step()
        out = jzt.check_lars_against_oracle(ps, got)
        assert out["flag"] == (1 if step == 2 else 0)
        ps.master_w, ps.momentum, ps.weight16 = got[0].copy(), got[1].copy(), got[2].copy()
