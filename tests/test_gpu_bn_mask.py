"""Batch normalization, the routes that depend on the workspace and on the tensor's size: the ReLU mask kept as bits between the
backward passes against the pass that reads y again, forward statistics with few, shared slabs against the oracle and in
their accuracy."""
import numpy as np
import pytest
import torch

import jzt
from paper_1807_11205_amd import inputs
from test_gpu_bn import _inputs, _run, jz  # noqa: F401

pytestmark = pytest.mark.gpu
# rows, channels: one word a lane and less, rows that end inside a group, several workgroups a slab, idle lanes
SHAPES = [(4160, 256), (12544, 72), (12545, 128), (3136, 2048), (3139, 1024), (70001, 8), (8192 + 3, 264)]


@pytest.mark.parametrize("rows,C", SHAPES)
def test_mask_words_give_the_bits_of_the_pass_over_y(jz, rows, C):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(rows + C)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    x, dy, y = rnd(rows, C).half(), rnd(rows, C).half(), rnd(rows, C).half()
    y.view(-1)[::7] = 0.0
    y.view(-1)[3::11] = float("nan")
    gamma, mean, invstd = rnd(C), rnd(C), rnd(C).abs() + 0.1
    full = jz.jz_bn_workspace_bytes(rows, C)
    res = []
    for n in (full, full - rows * C // 8):  # without room for the bits
        dx = torch.full((rows, C), 7.0, device="cuda", dtype=torch.float16)
        dg, db = torch.zeros(C, device="cuda", dtype=torch.float16), torch.zeros(C, device="cuda", dtype=torch.float16)
        ws = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        jz.jz_bn_relu_bwd(rows, C, x, y, dy, gamma, mean, invstd, True, dx, dg, db, ws[:n])
        assert bool((ws[n:] == 0xA5).all())
        res.append([jzt.bits(t.cpu().numpy()) for t in (dx, dg, db)])
    for a, b in zip(*res):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("tail", ["x", "y", "dy", "dx", "gamma", "mean", "invstd", "dg", "db"])
def test_a_tensor_of_the_call_behind_the_workspace_it_needs(jz, tail):  # noqa: F811
    """One piece of memory is passed as the workspace, and where the mask's bits would go lies a tensor of the call."""
    rows, C = 4160, 256                                 # 130 slabs: a workspace of 266240 + 4096 bytes and 133120 of bits
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    half, zero = torch.float16, lambda dt: torch.zeros(C, device="cuda", dtype=dt)
    t = dict(x=rnd(rows, C).half(), y=rnd(rows, C).half(), dy=rnd(rows, C).half(), dx=torch.zeros(rows, C, device="cuda", dtype=half),
             gamma=rnd(C), mean=rnd(C), invstd=rnd(C).abs() + 0.1, dg=zero(half), db=zero(half))
    full = jz.jz_bn_workspace_bytes(rows, C)
    need = 266240 + 4096
    assert full == need + 133120

    def call(ws, **o):
        a = dict(t, **o)
        jz.jz_bn_relu_bwd(rows, C, a["x"], a["y"], a["dy"], a["gamma"], a["mean"], a["invstd"], True, a["dx"], a["dg"], a["db"], ws)
        return [jzt.bits(a[k].cpu().numpy()) for k in ("dx", "dg", "db")]

    want = call(torch.zeros(full, dtype=torch.uint8, device="cuda"))
    n = t[tail].numel() * t[tail].element_size()
    memory = torch.zeros(max(full, need + n), dtype=torch.uint8, device="cuda")
    there = memory[need:need + n].view(t[tail].dtype).view(t[tail].shape)
    there.copy_(t[tail])
    for a, b in zip(call(memory, **{tail: there}), want):
        assert np.array_equal(a, b)


# sizes on either side of the limits of the shared-slab plan, channel counts that are not multiples of its 64
@pytest.mark.parametrize("rows,C", [(8191, 256), (8192, 256), (12545, 256), (3136, 2048), (29128, 72), (2100, 1000), (16385, 136)])
@pytest.mark.parametrize("relu", [True, False])
def test_forward_and_backward_against_the_oracle(jz, rows, C, relu):  # noqa: F811
    _run(jz, *_inputs((rows, C, 9), rows, C), 1e-5, relu)


def test_variance_of_channels_far_from_zero(jz):  # noqa: F811
    """Slabs of 128 rows shared by workgroups: the sums of squares are rounded to FP32 once a slab, 98 times in all, each time by
    at most 2^-24 (root mean square 3^-0.5 of that) of 101 variances, and invstd, whose relative error is half the variance's, once.  The
    factor allows for the spread of 256 channels."""
    rows, C = 12544, 256
    x = (inputs.rng_for(95, 1).standard_normal((rows, C), dtype=np.float32) + np.float32(10)).astype(np.float16)
    X = torch.from_numpy(x).cuda()
    one, y = torch.ones(C, device="cuda"), torch.empty_like(X)
    mean, invstd = torch.empty_like(one), torch.empty_like(one)
    jz.jz_bn_relu_fwd(rows, C, X, one, one, 0.0, False, y, mean, invstd, torch.zeros(jz.jz_bn_workspace_bytes(rows, C), dtype=torch.uint8, device="cuda"))
    want = 1.0 / x.astype(np.float64).std(0)
    err = float(np.sqrt(np.mean((invstd.cpu().numpy().astype(np.float64) / want - 1) ** 2)))
    assert err <= 1.2 * 2.0 ** -24 / 3 ** 0.5 * ((0.5 * 101 / 98 ** 0.5) ** 2 + 1) ** 0.5, err
