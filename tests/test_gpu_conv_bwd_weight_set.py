"""GPU parity of jz_conv2d_bwd_weight_set: sets of every size with members that end inside tiles, that split and that do not,
that run alone (3 channels, channel counts that are not multiples of 8), with the workspace it asks for, with less, and with
none."""
import numpy as np
import pytest
import torch

import oracle
from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu

# N, H, C, K, R, stride, pad
SETS = {
    "one": [(2, 9, 16, 24, 3, 1, 1)],
    "short": [(8, 2, 512, 2048, 1, 1, 0), (8, 2, 512, 512, 3, 1, 1), (8, 2, 1024, 2048, 1, 1, 0), (8, 1, 2048, 1000, 1, 1, 0)],
    "mixed": [(5, 13, 72, 136, 3, 1, 1), (3, 15, 64, 8, 1, 2, 0), (8, 16, 64, 64, 3, 1, 1), (4, 32, 3, 64, 7, 2, 3), (6, 11, 37, 50, 3, 1, 1),
              (2, 5, 8, 8, 5, 2, 2), (7, 9, 264, 40, 1, 1, 0), (1, 1, 8, 16, 1, 1, 0), (9, 14, 128, 256, 3, 2, 1), (2, 30, 24, 72, 1, 1, 0),
              (64, 7, 128, 128, 3, 1, 1)],
    "long": [(16, 28, 128, 128, 3, 1, 1), (16, 28, 128, 512, 1, 1, 0), (32, 14, 256, 256, 3, 1, 1)],
}


@pytest.mark.parametrize("name", SETS)
def test_set_against_the_oracle(name):
    import jzt
    from paper_1807_11205_amd import api as jz
    cases = [inputs.conv_case((4, i, *c), c[0], c[1], c[1], c[2], c[3], c[4], c[4], c[5], c[6], loss_scale=16.0, dy_std=0.05) for i, c in enumerate(SETS[name])]
    descs = [jzt.desc_of(c) for c in cases]
    x, dy = [jzt.to_dev(c.x) for c in cases], [jzt.to_dev(c.dy) for c in cases]
    want = [(oracle.conv_bwd_weight(jzt.odesc_of(c), c.x, c.dy), oracle.conv_bwd_weight(jzt.odesc_of(c), jzt.abs16(c.x), jzt.abs16(c.dy))) for c in cases]
    need = jz.jz_conv2d_bwd_weight_set_workspace_bytes(descs)
    # what members that run alone cannot do without (the 3-channel layer's padded copy)
    least = max((jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_WEIGHT, d) for d in descs if d.C % 8), default=0)
    for n in sorted({need, (need + least) // 2 // 256 * 256, least}):
        ws = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        dw = [torch.full((d.K, d.R, d.S, d.C), float("nan"), dtype=torch.float16, device="cuda") for d in descs]
        bound = jz.bind_conv2d_bwd_weight_set(descs, x, dy, dw, ws[:n] if n else None)
        bound()
        torch.cuda.synchronize()
        assert bool((ws[n:] == 0xA5).all())
        first = [t.cpu().numpy() for t in dw]
        for g, (ref, mag), c in zip(first, want, SETS[name]):
            jzt.check_half_output(g, ref, what="dw %s, %d bytes" % (c, n), mag64=mag)
        bound()
        torch.cuda.synchronize()
        assert all(np.array_equal(jzt.bits(a), jzt.bits(t.cpu().numpy())) for a, t in zip(first, dw))


# sets whose partial sums, added up in megabytes as floating-point numbers, come to more than the bytes that they are
ROUNDED = [[(13, 7, 136, 16, 3, 1, 1), (13, 7, 288, 216, 3, 1, 1), (23, 30, 8, 232, 1, 1, 0)], [(13, 30, 296, 112, 1, 1, 0)], [(19, 30, 192, 248, 3, 1, 1)],
           [(8, 28, 144, 112, 1, 1, 0), (15, 13, 176, 96, 3, 1, 1), (21, 7, 184, 96, 1, 1, 0), (6, 13, 184, 312, 3, 1, 1)]]


@pytest.mark.parametrize("layers", ROUNDED + [SETS["mixed"]], ids=lambda c: str(len(c)))
def test_the_reported_workspace_is_enough_for_the_reported_plan(layers):
    from paper_1807_11205_amd import api as jz
    descs = [jz.conv_desc(n, h, h, c, k, r, r, st, pad) for n, h, c, k, r, st, pad in layers]
    gen = torch.Generator(device="cuda").manual_seed(len(layers))
    rnd = lambda n: torch.randn(n, generator=gen, device="cuda").half()
    x, dy = [rnd(d.N * d.H * d.W * d.C) for d in descs], [rnd(d.N * d.P * d.Q * d.K) for d in descs]
    need, res = jz.jz_conv2d_bwd_weight_set_workspace_bytes(descs), []
    for more in (0, 1 << 20):                                   # with fewer splits the sums have another order
        dw = [torch.zeros(d.K * d.R * d.S * d.C, dtype=torch.float16, device="cuda") for d in descs]
        jz.jz_conv2d_bwd_weight_set(descs, x, dy, dw, torch.zeros(need + more, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        res.append(torch.cat(dw).view(torch.int16))
    assert torch.equal(*res)


def test_argument_errors():
    from paper_1807_11205_amd import api as jz
    d = jz.conv_desc(4, 8, 8, 16, 16, 3, 3, 1, 1)
    x, dy = (torch.zeros(4 * 8 * 8 * 16, dtype=torch.float16, device="cuda") for _ in range(2))
    dw = [torch.zeros(16 * 9 * 16, dtype=torch.float16, device="cuda") for _ in range(2)]
    bind = lambda w: jz.bind_conv2d_bwd_weight_set([d, d], [x, x], [dy, dy], w, torch.zeros(1 << 20, dtype=torch.uint8, device="cuda"))
    bind(dw)()
    with pytest.raises(jz.JzError):
        bind([dw[0], dw[0]])()                      # two results in one place
    with pytest.raises(jz.JzError):
        bind([dw[0], x[:dw[0].numel()]])()          # a result over an operand
    with pytest.raises(jz.JzError):
        jz.jz_conv2d_bwd_weight_set_workspace_bytes([d] * 12)
    torch.cuda.synchronize()
