"""Pooling kernels at the edges of their cells and grids against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1807_11205_amd import inputs

pytestmark = pytest.mark.gpu

# N, H, W, C, window, stride, pad: 3 x 3 with stride 2 goes by cells of 2 x 2 positions, which start before the image without padding and
# end behind it for either parity of the size; then the general gather, more images than a grid dimension takes, and rows that share a workgroup (of
# 4, 49 and 128 threads, forward, the last of them not all there) or just do not (129)
POOLS = [(2, 3, 3, 8, 3, 2, 0), (3, 7, 10, 8, 3, 2, 1), (2, 6, 5, 24, 3, 2, 2), (1, 1, 2, 8, 3, 2, 1), (2, 8, 9, 16, 3, 2, 0), (2, 9, 8, 16, 3, 1, 1),
         (65537, 3, 3, 8, 3, 2, 1), (4097, 4, 8, 8, 2, 2, 0), (301, 7, 7, 56, 3, 1, 1), (3, 30, 32, 64, 3, 2, 1), (2, 9, 86, 24, 2, 2, 0)]


@pytest.mark.parametrize("N,H,W,C,window,stride,pad", POOLS)
def test_pool_edges(N, H, W, C, window, stride, pad):
    from paper_1807_11205_amd import api
    rng = inputs.rng_for(77, N, H, W, C, stride, pad)
    n = min(N, 3)                      # the oracle loops over images: the first and the last ones
    x = (rng.integers(-4, 5, size=(N, H, W, C)) * 0.5).astype(np.float16)       # ties
    P, Q = oracle.pool_out(H, window, stride, pad), oracle.pool_out(W, window, stride, pad)
    dy = rng.standard_normal((N, P, Q, C), dtype=np.float32).astype(np.float16)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).ravel()).cuda()
    y, dx, dx2 = (torch.full((k,), 9.0, dtype=torch.float16, device="cuda") for k in (N * P * Q * C, x.size, x.size))
    arg = torch.zeros(N * P * Q * C, dtype=torch.uint8, device="cuda")
    tx, tdy = dev(x), dev(dy)
    api.jz_maxpool_fwd(N, H, W, C, window, stride, pad, tx, y, arg)
    api.jz_maxpool_bwd(N, H, W, C, window, stride, pad, None, tdy, dx, arg)
    api.jz_maxpool_bwd(N, H, W, C, window, stride, pad, tx, tdy, dx2)
    torch.cuda.synchronize()
    assert torch.equal(dx.view(torch.int16), dx2.view(torch.int16))              # with and without the saved winners
    for part in (slice(0, n), slice(N - n, N)):
        ry, rarg = oracle.maxpool_fwd(x[part], window, stride, pad)
        assert np.array_equal(y.cpu().numpy().reshape(N, P, Q, C)[part].view(np.uint16), ry.reshape(-1, P, Q, C).view(np.uint16))
        _, r16 = oracle.maxpool_bwd(x[part], dy[part], window, stride, pad)
        got = dx.cpu().numpy().reshape(N, H, W, C)[part].astype(np.float64)
        assert np.all(np.abs(got - np.asarray(r16, np.float64).reshape(got.shape)) <= 2.0 ** -10 * np.abs(got) + 2.0 ** -24)


@pytest.mark.skipif(torch.cuda.is_available() and torch.cuda.mem_get_info()[0] < 100 << 30, reason="needs 70 GB of device memory")
def test_a_row_of_more_than_32_bits():
    """2^20 + 1 positions of 4096 x 8 channels: more threads than a dimension of a grid counts."""
    from paper_1807_11205_amd import api
    W, C, stride = (1 << 20) + 1, 32768, 64
    Q = (W - 1) // stride + 1
    dy = torch.randn(Q * C // 64, device="cuda").half().repeat(64)
    arg = torch.zeros(Q * C, dtype=torch.uint8, device="cuda")
    dx = torch.empty(W * C, dtype=torch.float16, device="cuda")
    for w in (0, 1, W - 2, W - 1):
        dx[w * C:(w + 1) * C] = 7.0
    api.jz_maxpool_bwd(1, 1, W, C, 1, stride, 0, None, dy, dx, arg)
    torch.cuda.synchronize()
    for w in (0, 1, W - 2, W - 1):
        want = dy[w // stride * C:(w // stride + 1) * C] if w % stride == 0 else torch.zeros(C, dtype=torch.float16, device="cuda")
        assert torch.equal(dx[w * C:(w + 1) * C], want), w
    del dx, dy, arg
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,HW,C", [(1, 1, 8), (2, 5, 16), (3, 15, 24), (2, 16, 520), (5, 17, 8), (2, 49, 2048)])
def test_average_pool_edges(N, HW, C):
    from paper_1807_11205_amd import api
    rng = inputs.rng_for(78, N, HW, C)
    x = rng.standard_normal((N, HW, 1, C), dtype=np.float32).astype(np.float16)
    y = torch.empty(N * C, dtype=torch.float16, device="cuda")
    api.jz_avgpool_fwd(N, HW, C, torch.from_numpy(x.ravel()).cuda(), y)
    acc = np.zeros((N, C), np.float32)                                            # FP32, in order: the same bits
    for j in range(HW):
        acc += x[:, j, 0].astype(np.float32)
    assert np.array_equal(y.cpu().numpy().reshape(N, C).view(np.uint16), (acc / np.float32(HW)).astype(np.float16).view(np.uint16))
