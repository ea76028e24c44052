"""Batch normalization of a whole tensor in one launch (channel counts that are multiples of 64): the edges of what a workgroup keeps, against
formulas in FP64; the same bits as the launches apart (which a captured graph takes) and when workgroups end without their rows written."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture()
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    assert torch.cuda.is_available()
    c = Case(api, 512, 64)
    o = c.outputs()
    for _ in range(66):            # one stream a device runs it in one launch: the one that called last, and often
        c.forward(o)
    assert _in_one_launch(c, lambda: c.forward(o))
    yield api
    api.jz_bn_tune_wait(10)


class Case:
    def __init__(self, jz, rows, C, seed=0):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(1000 * C + rows + seed)
        rn = lambda n, std, dt, mean=0.0: (torch.randn(n, generator=gen, device=DEV) * std + mean).to(dt)
        h, f = torch.float16, torch.float32
        self.jz, self.rows, self.C = jz, rows, C
        n = rows * C
        self.x, self.dy, self.dy2 = rn(n, 1.5, h, 0.3), rn(n, 1.0, h), rn(n, 1.0, h)
        self.gamma, self.beta = rn(C, 0.1, f, 1.0), rn(C, 0.1, f)
        self.ws = torch.empty(jz.jz_bn_workspace_bytes(rows, C), dtype=torch.uint8, device=DEV)

    def outputs(self, fill=7.0):
        n, C = self.rows * self.C, self.C
        h = lambda k: torch.full((k,), fill, dtype=torch.float16, device=DEV)
        f = lambda k: torch.full((k,), fill, dtype=torch.float32, device=DEV)
        return dict(y=h(n), mean=f(C), invstd=f(C), dx=h(n), dg=h(C), db=h(C), dx0=h(n), dg0=h(C), db0=h(C), g=h(n), dxe=h(n), dge=h(C), dbe=h(C))

    def forward(self, o):
        self.jz.jz_bn_relu_fwd(self.rows, self.C, self.x, self.gamma, self.beta, 1e-5, True, o["y"], o["mean"], o["invstd"], self.ws)

    def run(self, o):
        jz, r, c = self.jz, self.rows, self.C
        self.forward(o)
        jz.jz_bn_relu_bwd(r, c, self.x, o["y"], self.dy, self.gamma, o["mean"], o["invstd"], True, o["dx"], o["dg"], o["db"], self.ws)
        jz.jz_bn_relu_bwd(r, c, self.x, None, self.dy, self.gamma, o["mean"], o["invstd"], False, o["dx0"], o["dg0"], o["db0"], self.ws)
        jz.jz_bn_bwd_block_end(r, c, self.x, o["y"], self.dy, self.dy2, self.gamma, o["mean"], o["invstd"], o["g"], o["dxe"], o["dge"], o["dbe"], self.ws)


def _plan(rows, C):
    """Slabs and groups of channels of the one launch."""
    groups, least = C // 64, 256 if rows <= 256 or rows >= 4096 else 128
    return -(-rows // max(least, -(-rows // (256 // groups)))), groups


def _in_one_launch(c, call):
    """Whether a call ran in one launch: it leaves the launch's tag and "sums are there" (2) in a word for every workgroup behind the slabs' FP64 sums."""
    slabs, groups = _plan(c.rows, c.C)
    assert slabs > 1, "workgroups that wait for nobody leave no flags"
    at = (slabs * 2 * c.C * 8 + 255) // 256 * 256
    c.ws.fill_(0xCD)
    torch.cuda.synchronize()
    call()
    torch.cuda.synchronize()
    words = c.ws[at:at + 8 * slabs * groups].view(torch.int64)
    return bool((words == words[0]).all()) and int(words[0]) & 3 == 2


def _same(a, b):
    bits = lambda t: t.view(torch.int16 if t.element_size() == 2 else torch.int32)
    return {k: int((bits(a[k]) != bits(b[k])).sum()) for k in a if not torch.equal(bits(a[k]), bits(b[k]))}


def _rel(a, ref):
    return float((a.double() - ref).norm() / ref.norm().clamp_min(1e-30))


def _check(c, o):
    """FP16 results within one rounding (2.8e-4 relative on average, 1e-3 allowed as everywhere); the statistics are FP32."""
    R, C = c.rows, c.C
    x = c.x.view(R, C).double()
    mean, var = x.mean(0), x.var(0, unbiased=False)
    inv = 1.0 / torch.sqrt(var + 1e-5)
    assert float(((o["mean"].double() - mean).abs() * inv).max()) <= 1e-5
    assert float(((o["invstd"].double() - inv) / inv).abs().max()) <= 1e-4
    y = torch.relu((x - mean) * inv * c.gamma.double() + c.beta.double())
    assert _rel(o["y"].view(R, C), y) <= 1e-3
    xh = (x - o["mean"].double()) * o["invstd"].double()
    del y, x
    zero = torch.zeros((), dtype=torch.float64, device=DEV)
    keep = o["y"].view(R, C) > 0
    dy = c.dy.view(R, C).double()
    both = (c.dy.view(R, C).float() + c.dy2.view(R, C).float()).half().double()
    for g, dx, dg, db in ((torch.where(keep, dy, zero), "dx", "dg", "db"), (dy, "dx0", "dg0", "db0"), (torch.where(keep, both, zero), "dxe", "dge", "dbe")):
        sb, sg = g.sum(0), (g * xh).sum(0)
        ref = c.gamma.double() * o["invstd"].double() * (g - sb / R - xh * (sg / R))
        # one rounding, and where the difference cancels (few rows) what FP32 leaves of gamma invstd g
        assert float((o[dx].view(R, C).double() - ref).norm()) <= 1e-3 * float(ref.norm()) + 1e-6 * float((c.gamma.double() * o["invstd"].double() * g).norm()), dx
        floor = R ** 0.5 * 1e-2
        for got, want in ((o[dg], sg), (o[db], sb)):
            assert float(((got.double() - want).abs() / want.abs().clamp_min(floor)).max()) <= 2e-3
    assert torch.equal(o["g"].view(R, C).double(), torch.where(keep, both, zero))


def _graph_run(c, o):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run(o)
    torch.cuda.current_stream().wait_stream(s)
    for _ in range(3):
        c.ws.fill_(0xCD)
        g.replay()
        torch.cuda.synchronize()


# 256 workgroups of 64 channels each, a pass of 64 rows: rows = passes * 64 * 256 / (C / 64) fill the chip
FULL = [(p * 64 * (256 // (C // 64)), C) for p, C in ((4, 2048), (8, 1024), (14, 512), (25, 256))]
SIZES = [(1, 64), (63, 64), (64, 128), (65, 64), (129, 2048), (1000, 192), (777, 320), (4099, 1984),
         (49, 2048), (64, 1024), (256, 64),     # one workgroup has all rows of its channels: its wavefronts wait for each other's sums
         (257, 64), (4095, 64), (4097, 64),     # two of 128 rows, 32, 17 of 256
         (8193, 64), (16384, 64), (16385, 64)]  # 33 slabs: more than one for a lane; 64: the launches apart merge them, 65: they do not
SIZES += [(r + d, C) for r, C in FULL for d in (0, 1)]


@pytest.mark.parametrize("rows,C", SIZES)
def test_edges(jz, rows, C):
    c = Case(jz, rows, C)
    a, b = c.outputs(), c.outputs()
    c.ws.fill_(0xCD)
    if _plan(rows, C)[0] > 1:
        assert _in_one_launch(c, lambda: c.run(a))
    else:
        c.run(a)
        torch.cuda.synchronize()
    _check(c, a)
    _graph_run(c, b)
    assert _same(a, b) == {}
    jz.jz_bn_tune_wait(0)          # nobody waits: whoever is first takes rows over
    try:
        for _ in range(3):
            b = c.outputs(fill=-3.0)
            c.ws.fill_(0xCD)
            c.run(b)
            torch.cuda.synchronize()
            assert _same(a, b) == {}
    finally:
        jz.jz_bn_tune_wait(10)


@pytest.mark.parametrize("passes", [33, 43, 44, 46, 47, 80, 81, 82])   # forward keeps 43, backward 25, and the bits of 56 beyond 24
def test_more_rows_than_are_kept(jz, passes):
    c = Case(jz, passes * 64 * 64 - 5, 256)
    a, b = c.outputs(), c.outputs()
    assert _in_one_launch(c, lambda: c.run(a))
    _check(c, a)
    _graph_run(c, b)
    assert _same(a, b) == {}
    jz.jz_bn_tune_wait(0)
    try:
        b = c.outputs(fill=-3.0)
        c.run(b)
        torch.cuda.synchronize()
        assert _same(a, b) == {}
    finally:
        jz.jz_bn_tune_wait(10)


@pytest.mark.parametrize("rows,C", [(784, 512), (3136, 256), (12544, 64)])
def test_sums_between_lanes_and_workgroups_are_fp64(jz, rows, C):
    """Large terms that cancel, in different workgroups, in lanes (a lane has every 64th row) that hold nothing else; the other terms are 2^-16.  Every
    lane's FP32 sum is exact and so is every FP64 sum of them, while FP32 sums at the size of the large terms (ulp 2^-9) lose the small ones."""
    t = torch.full((rows, C), 2.0 ** -16, device=DEV)
    t[0::64], t[1::64] = 0.0, 0.0
    t[0], t[1 + rows // 128 * 64] = 30000.0, -30000.0
    total = int((t == 2.0 ** -16).sum()) // C * 2.0 ** -16
    t = t.half().view(-1)
    c = Case(jz, rows, C)
    one, zero = torch.ones(C, device=DEV), torch.zeros(C, device=DEV)
    x = torch.ones(rows * C, dtype=torch.float16, device=DEV)

    def run(o):
        jz.jz_bn_relu_fwd(rows, C, t, one, zero, 1e-5, False, o["y"], o["mean"], o["invstd"], c.ws)
        jz.jz_bn_relu_bwd(rows, C, x, x, t, one, zero, one, True, o["dx"], o["dg"], o["db"], c.ws)
        jz.jz_bn_relu_bwd(rows, C, x, None, t, one, zero, one, False, o["dx0"], o["dg0"], o["db0"], c.ws)
        jz.jz_bn_bwd_block_end(rows, C, x, x, t, None, one, zero, one, o["g"], o["dxe"], o["dge"], o["dbe"], c.ws)

    c.run = run
    o, b = c.outputs(), c.outputs()
    run(o)
    torch.cuda.synchronize()
    mean = torch.tensor(total * (1.0 / rows), dtype=torch.float64)
    assert float((o["mean"].double().cpu() / mean - 1).abs().max()) <= 2.0 ** -24
    for k in ("dg", "db", "dg0", "db0", "dge", "dbe"):
        assert torch.equal(o[k], torch.full_like(o[k], total)), (k, o[k][:2], total)
    _graph_run(c, b)
    assert _same(o, b) == {}


@pytest.mark.parametrize("rows,C", [(802816, 64), (200704 - 37, 256), (50176, 512)])
def test_beside_a_kernel_that_holds_a_compute_unit(jz, rows, C):
    """Tensors that need all compute units, while another stream's kernel has one for 20 ms: the rows of the workgroup that cannot start are taken over, with
    the same bits, and long before that kernel ends.  The bound is ten times the slowest of these calls; waiting for the absent workgroup or leaving it the
    others' rows took 1 to 20 ms."""
    c = Case(jz, rows, C)
    a, b = c.outputs(), c.outputs()
    c.run(a)
    side, ev = torch.cuda.Stream(), lambda: torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t = ev(), ev()
    t[0].record()
    torch.cuda._sleep(2000000)
    t[1].record()
    torch.cuda.synchronize()
    per_ms = 2000000 / t[0].elapsed_time(t[1])
    with torch.cuda.stream(side):
        torch.cuda._sleep(int(20 * per_ms))
    torch.cuda._sleep(int(0.1 * per_ms))          # the other one has started
    t = ev(), ev()
    t[0].record()
    c.run(b)
    t[1].record()
    t[1].synchronize()
    held = not side.query()
    torch.cuda.synchronize()
    assert _same(a, b) == {}
    assert held and t[0].elapsed_time(t[1]) <= 10 * 4 * 0.25, t[0].elapsed_time(t[1])


def test_several_streams_at_once(jz):
    cases = [Case(jz, 20000 + 64 * i, 128, seed=i) for i in range(5)]
    want = [c.outputs() for c in cases]
    for c, o in zip(cases, want):
        c.run(o)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    for _ in range(4):
        got = [c.outputs() for c in cases]
        torch.cuda.synchronize()
        for _ in range(30):         # one of the streams has the one launch
            for c, o, s in zip(cases, got, streams):
                with torch.cuda.stream(s):
                    c.run(o)
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            assert _same(a, b) == {}
    got = [c.outputs() for c in cases]
    torch.cuda.synchronize()
    for c, o, s in zip(cases, got, streams):
        with torch.cuda.stream(s):
            for _ in range(18):     # 72 calls: it moves on to this stream while the work of the one before is on its way
                c.run(o)
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        assert _same(a, b) == {}
    with torch.cuda.stream(streams[-1]):
        assert _in_one_launch(cases[-1], lambda: cases[-1].run(got[-1]))


def test_a_stream_that_is_kept_to_half_of_the_compute_units(jz):
    """It never has the one launch, whose workgroups it could not run together."""
    import ctypes
    hip, stream = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, (ctypes.c_uint32 * 8)(*[0xffffffff] * 4, *[0] * 4)) == 0
    c = Case(jz, 50176, 128)
    a, b = c.outputs(), c.outputs()
    assert _in_one_launch(c, lambda: c.run(a))
    with torch.cuda.stream(torch.cuda.ExternalStream(stream.value)):
        for _ in range(70):
            c.run(b)
        torch.cuda.synchronize()
        assert not _in_one_launch(c, lambda: c.run(b))
    assert _same(a, b) == {}


def test_statistics_saved_over_the_parameters(jz):
    """Accepted where the statistics are finished in a launch of their own, which reads a channel's parameters before it writes there."""
    c = Case(jz, 200704, 64)
    a, b = c.outputs(), c.outputs()
    c.forward(a)
    c.gamma, c.beta, b["mean"], b["invstd"] = b["mean"].copy_(c.gamma), b["invstd"].copy_(c.beta), b["mean"], b["invstd"]
    assert not _in_one_launch(c, lambda: c.forward(b))
    assert float(((a["mean"] - b["mean"]) * a["invstd"]).abs().max()) <= 1e-5 and float((a["invstd"] / b["invstd"] - 1).abs().max()) <= 1e-5
    assert float((a["y"].float() - b["y"].float()).abs().max()) <= 2.0 ** -10 * float(a["y"].abs().max())     # one FP16 rounding the other way


@pytest.mark.parametrize("over", ["y over gamma, beta", "dx over gamma, mean, invstd", "block end's dx over them"])
def test_results_over_the_parameters(jz, over):
    """Accepted, and right where a launch of its own reads the parameters before results are written there (103 MB forward, 26 MB backward)."""
    forward = over[0] == "y"
    rows, C = (802816 if forward else 200704), 64
    c = Case(jz, rows, C)
    a, b = c.outputs(), c.outputs()
    c.run(a)
    out = "y" if forward else "dx" if over[0] == "d" else "dxe"
    words = b[out].view(torch.float32)
    at = [words[(rows // 3 + i) * 64:][:C] for i in range(3)]        # whole rows in the middle of the result
    if forward:
        c.gamma, c.beta = at[0].copy_(c.gamma), at[1].copy_(c.beta)
        call = lambda: c.forward(b)
    else:
        c.gamma, mean, invstd = at[0].copy_(c.gamma), at[1].copy_(a["mean"]), at[2].copy_(a["invstd"])
        if out == "dx":
            call = lambda: jz.jz_bn_relu_bwd(rows, C, c.x, a["y"], c.dy, c.gamma, mean, invstd, True, b["dx"], b["dg"], b["db"], c.ws)
        else:
            call = lambda: jz.jz_bn_bwd_block_end(rows, C, c.x, a["y"], c.dy, c.dy2, c.gamma, mean, invstd, b["g"], b["dxe"], b["dge"], b["dbe"], c.ws)
    assert not _in_one_launch(c, call)
    assert float((a[out].float() - b[out].float()).abs().max()) <= 2.0 ** -10 * float(a[out].abs().max())     # one FP16 rounding the other way


def test_infinities_and_nan_stay_in_their_channels(jz):
    c = Case(jz, 5000, 128)
    clean = c.outputs()
    c.run(clean)
    x = c.x.view(5000, 128)
    x[17, 3], x[4000, 70] = float("inf"), float("nan")
    o, b = c.outputs(), c.outputs()
    assert _in_one_launch(c, lambda: c.run(o))
    _graph_run(c, b)
    ok = [i for i in range(128) if i not in (3, 70)]
    for k in ("y", "dx", "dx0"):
        assert torch.equal(o[k].view(5000, 128)[:, ok], clean[k].view(5000, 128)[:, ok])
    for k in ("mean", "invstd", "dg", "db"):
        assert torch.equal(o[k][ok], clean[k][ok])
        assert torch.equal(torch.isfinite(o[k]), torch.isfinite(b[k]))
    assert not torch.isfinite(o["mean"][[3, 70]]).any()
