"""The binding's native part (no GPU): what it does not take for certain is left to the Python checks, which say what is wrong."""
import ctypes

import pytest
import torch

from paper_1807_11205_amd import _jz_host as host
from paper_1807_11205_amd import api


def test_tensors_that_are_not_plainly_in_order_are_left_alone():
    t = torch.zeros(8, dtype=torch.float16)
    for o in (t, t.to("meta"), None, 3, "x", torch.zeros(0, dtype=torch.float16)):
        assert host.ptr(o, torch.float16, 8) is None
        assert host.ws(o) is None
    assert host.ptr(t, "half", 8) is None and host.ptr(t, torch.float16, 1 << 80) is None and host.ptr(t, torch.float16, "8") is None
    with pytest.raises(TypeError, match="x16 must be a contiguous torch.float16 tensor on the GPU"):
        api._dev_ptr(t, torch.float16, 8, "x16")
    with pytest.raises(TypeError, match="workspace must be a contiguous GPU tensor"):
        api._ws(t)
    d = api.conv_desc(1, 4, 4, 8, 8, 3, 3, 1, 1)
    x, w = torch.zeros(128, dtype=torch.float16), torch.zeros(576, dtype=torch.float16)
    for desc in (d, api.conv_desc(1, 4, 4, 8, 8, 3, 3, 0, 1), api.conv_desc(1, 1, 1, 8, 8, 3, 3, 1, 0), api.conv_desc(1 << 30, 1 << 30, 1 << 30, 1 << 30, 8, 1, 1),
                 b"short", object()):
        assert host.conv(1, api.JZ_FWD, desc, x, w, x, None, torch.float16, 0, int) == host.LOOK      # 1: nothing is called
    assert host.conv(1, 7, d, x, w, x, None, torch.float16, 0, int) == host.LOOK
    for call, a in ((api.jz_conv2d_fwd, (x, w, x)), (api.jz_conv2d_bwd_data, (x, w, x)), (api.jz_conv2d_bwd_weight, (x, x, w))):
        with pytest.raises(TypeError, match="must be a contiguous"):
            call(d, *a)
        with pytest.raises(TypeError, match="ctypes instance"):     # the descriptor's bytes are not a descriptor
            call(bytes(d), *a)


def test_bound_calls_pass_every_kind_of_argument():
    """The same statuses as through ctypes, for argument lists of the shortest and of the longest entry points."""
    seen = []

    def record(*a):
        seen.append(a)
        return -7

    for n in (1, 2, 7, 15, 24):
        proto = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_int if i == 0 else ctypes.c_size_t for i in range(n + 1)])
        f = proto(record)
        args = (-5,) + tuple((1 << 63) + i for i in range(1, n))
        assert host.invoke(ctypes.cast(f, ctypes.c_void_p).value, args, 12345) == -7
        assert seen[-1] == args + (12345,)
    with pytest.raises(TypeError):
        host.invoke(0, tuple(range(25)), 0)
    d = api.conv_desc(1, 4, 4, 8, 8, 3, 3, 1, 1)
    arr = (ctypes.c_void_p * 3)(1, 2, 3)
    assert api._words((ctypes.byref(d), None, 7, arr)) == (ctypes.addressof(d), 0, 7, ctypes.addressof(arr))
    assert api._words((1, 0.5)) is None and api._words(tuple(range(25))) is None
    with pytest.raises(api.JzError):        # a null output, found by the library
        api.BoundCall(api.lib().jz_conv2d_fwd, (ctypes.byref(d), 16, 32, None, None, 0), "jz_conv2d_fwd", (d,))(0)


def test_the_binding_can_be_imported_before_anything_is_built(tmp_path):
    """Descriptors, status names and shapes need no native code; the first call that does says what is missing."""
    import shutil
    import subprocess
    import sys
    import paper_1807_11205_amd
    src = paper_1807_11205_amd.__path__[0]
    shutil.copytree(src, tmp_path / "paper_1807_11205_amd", ignore=shutil.ignore_patterns("*.so", "__pycache__", "csrc"))
    code = ("import ctypes, torch\nfrom paper_1807_11205_amd import api, shapes, tune\nd = api.conv_desc(1, 8, 8, 16, 16, 3, 3, 1, 1)\n"
            "assert d.P == 8 and shapes.resnet50_convs()\ntry:\n    api._dev_ptr(torch.zeros(1), torch.float32)\nexcept ImportError:\n    print('missing')\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "missing", out.stderr
