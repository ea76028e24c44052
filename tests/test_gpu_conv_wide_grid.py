"""Images of more than 2^23 columns or rows: pixel coordinates beyond 24 bits, in the masks of padding taps and in the gathered
operand of the weight gradient.  Operands are zero but for the first and the last few hundred pixels, so that a pixel that
drops out shows; the expected values are FP64 sums over those.
Tolerance: FP16 inputs N(0,1) with K <= 64 products per output, FP32 accumulation (1e-6) and one FP16 rounding (2^-11): 1e-3 of
the result's norm; weight gradients add up to 1024 products per element, the same bound; FP32: 1024 * 2^-24 < 1e-4."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LONG, END = (1 << 23) + 1200, 500


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    assert torch.cuda.is_available()
    return api


def run_case(jz, half, C, K, S, stride, pad, vertical, ops):
    dt = torch.float16 if half else torch.float32
    Q = LONG
    W = (Q - 1) * stride + S - 2 * pad
    d = (jz.conv_desc(1, W, 1, C, K, S, 1, (stride, 1), (pad, 0)) if vertical else jz.conv_desc(1, 1, W, C, K, 1, S, (1, stride), (0, pad)))
    assert max(d.P, d.Q) == Q
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *n: torch.randn(*n, generator=g, device="cuda").to(dt)
    x, dy = torch.zeros(W, C, dtype=dt, device="cuda"), torch.zeros(Q, K, dtype=dt, device="cuda")
    for t, n in ((x, END * stride), (dy, END)):
        t[:n] = rand(n, t.shape[1])
        t[-n:] = rand(n, t.shape[1])
    w = rand(K, S, C)
    bind, need = (jz.bind_conv2d, jz.jz_conv2d_workspace_bytes) if half else (jz.bind_conv2d_f32, jz.jz_conv2d_f32_workspace_bytes)
    tol = 1e-3 if half else 1e-4
    x64, dy64, w64 = x.cpu().double().numpy(), dy.cpu().double().numpy(), w.cpu().double().numpy()

    def call(op, a, b, out):
        ws = torch.empty(max(need(op, d), 16), dtype=torch.uint8, device="cuda")
        bind(op, d, a, b, out, ws)()
        torch.cuda.synchronize()
        return out

    def close(got, want, what):
        got = got.double().cpu().numpy()
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print(what, "%.2e" % err, flush=True)
        assert err < tol, (what, err)

    ends = lambda n, m: np.r_[0:m, n - m:n]
    if "fwd" in ops:
        y = call(jz.JZ_FWD, x, w, torch.full((Q, K), float("nan"), dtype=dt, device="cuda"))
        q = ends(Q, END // 2)
        want = np.zeros((len(q), K))
        for s in range(S):
            i = q * stride - pad + s
            ok = (i >= 0) & (i < W)
            want[ok] += x64[i[ok]] @ w64[:, s].T
        close(y[torch.as_tensor(q, device="cuda")], want, "fwd")
        assert not y[END + S:-END - S].any()          # zero where the operand is, none left unwritten
    if "bwd_data" in ops:
        dx = call(jz.JZ_BWD_DATA, dy, w, torch.full((W, C), float("nan"), dtype=dt, device="cuda"))
        h = ends(W, END // 2)
        want = np.zeros((len(h), C))
        for s in range(S):
            q, rem = np.divmod(h + pad - s, stride)
            ok = (rem == 0) & (q >= 0) & (q < Q)
            want[ok] += dy64[q[ok]] @ w64[:, s]
        close(dx[torch.as_tensor(h, device="cuda")], want, "bwd_data")
    if "bwd_weight" in ops:
        dw = call(jz.JZ_BWD_WEIGHT, x, dy, torch.full((K, S, C), float("nan"), dtype=dt, device="cuda"))
        want = np.zeros((K, S, C))
        for s in range(S):
            q = ends(Q, END)
            i = q * stride - pad + s
            ok = (i >= 0) & (i < W)
            want[:, s] = dy64[q[ok]].T @ x64[i[ok]]
        close(dw, want, "bwd_weight")


ALL = ("fwd", "bwd_data", "bwd_weight")
CASES = [
    # half, C, K, S, stride, pad, along the rows, operations
    (True, 8, 8, 3, 1, 1, False, ALL),            # flattened taps; masks
    (True, 8, 8, 3, 1, 1, True, ALL),
    (True, 32, 8, 3, 1, 1, False, ("fwd", "bwd_weight")),
    (True, 8, 8, 2, 2, 0, False, ALL),            # strided: the residues of the stride
    (True, 8, 8, 3, 1, 0, True, ("bwd_data", "bwd_weight")),
    (False, 4, 4, 3, 1, 0, False, ALL),           # gathered x with a grid of another size
    (False, 4, 4, 3, 1, 1, True, ALL),            # ... of the same size
    (False, 4, 4, 2, 2, 0, True, ALL),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%d_%d_%dtap_s%d_p%d_%s" % ("f16" if c[0] else "f32", *c[1:6], "rows" if c[6] else "cols"))
def test_more_than_2_to_23_pixels_along_one_axis(jz, case):
    run_case(jz, *case)
