"""Two threads, each on a stream of its own, running convolutions of both precisions at the same time: first launches (kernel
attributes, plans) included, the bits are those of one thread."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LAYERS = [(2, 14, 16, 16, 3, 1), (3, 15, 40, 72, 3, 2), (4, 28, 64, 128, 3, 1), (5, 14, 256, 64, 1, 1), (2, 30, 3, 64, 7, 2), (3, 9, 37, 50, 3, 1),
          (4, 13, 64, 64, 3, 2), (2, 16, 128, 256, 1, 2)]


def run_layers(jz, order, out):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for i in order:
            N, H, C, K, R, st = LAYERS[i]
            d = jz.conv_desc(N, H, H, C, K, R, R, st, R // 2)
            g = torch.Generator(device="cuda").manual_seed(i)
            x, w, dy = (torch.randn(n, generator=g, device="cuda") for n in (N * H * H * C, K * R * R * C, N * d.P * d.Q * K))
            for f32 in (True, False):
                dt = torch.float32 if f32 else torch.float16
                bind, need = (jz.bind_conv2d_f32, jz.jz_conv2d_f32_workspace_bytes) if f32 else (jz.bind_conv2d, jz.jz_conv2d_workspace_bytes)
                t = {k: v.to(dt) for k, v in dict(x=x, w=w, dy=dy).items()}
                for op, a, b, like in ((jz.JZ_FWD, "x", "w", "dy"), (jz.JZ_BWD_DATA, "dy", "w", "x"), (jz.JZ_BWD_WEIGHT, "x", "dy", "w")):
                    y = torch.full_like(t[like], float("nan"))
                    ws = torch.empty(max(16, need(op, d)), dtype=torch.uint8, device="cuda")
                    bind(op, d, t[a], t[b], y, ws)(stream)
                    out[i, f32, op] = y.cpu().numpy()         # waits for the stream


def test_convolutions_on_two_threads():
    from paper_1807_11205_amd import api as jz
    jz.lib()
    got = [{}, {}]
    n = len(LAYERS)
    threads = [threading.Thread(target=run_layers, args=(jz, order, out)) for order, out in ((range(n), got[0]), (range(n - 1, -1, -1), got[1]))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    alone = {}
    run_layers(jz, range(n), alone)
    assert len(alone) == 6 * n
    for k, v in alone.items():
        assert not np.isnan(v).any()
        for g in got:
            assert np.array_equal(v.view(np.uint8), g[k].view(np.uint8)), k
