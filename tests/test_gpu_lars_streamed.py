"""GPU parity of the LARS update on either side of 2^25 parameters, where weights and momentum no longer fit the last-level cache
and are read with the non-temporal hint: both update paths, a second tensor that starts off every 16-byte boundary, a fresh
workspace and carried sums of the weights."""
import numpy as np
import pytest
import torch

from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu

LIMIT = 1 << 25


@pytest.mark.parametrize("path", ["three_launches", "presummed"])
@pytest.mark.parametrize("total", [LIMIT, LIMIT + 1, LIMIT + 70001])
def test_two_steps_against_the_oracle(path, total):
    import jzt
    assert torch.cuda.is_available()
    sizes = [20000003, total - 20000003 - 9, 9]
    ps = inputs.random_param_set((0, 79, total % 1000), sizes, loss_scale=256.0, momentum_std=1e-3, flags=[3, 1, 2])
    r = jzt.LarsRun(ps, path=path)
    for step in range(2):
        got = r.step()
        out = jzt.check_lars_against_oracle(ps, got)
        print("step", step, out, flush=True)
        ps.master_w, ps.momentum, ps.weight16 = got[0].copy(), got[1].copy(), got[2].copy()
