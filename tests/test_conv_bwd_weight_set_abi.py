"""jz_conv2d_bwd_weight_set refuses a call before its first launch, whichever member is at fault: those that share a launch and
those that run alone (channel counts that are not multiples of 8, 3-channel stems).  Host only: addresses are never used."""
import ctypes
import weakref

import pytest
import torch

from paper_1807_11205_amd import api

A = 0x10000000
STEP = 0x1000000
STEM, ODD, FAST = (4, 32, 32, 3, 64, 7, 7, 2, 3), (6, 11, 11, 37, 50, 3, 3, 1, 1), (2, 8, 8, 16, 16, 3, 3, 1, 1)


def call(layers, ws_bytes=1 << 22, **at):
    n = len(layers)
    descs = (api.jz_conv_desc * n)(*(api.conv_desc(*c) for c in layers))
    arr = ctypes.c_void_p * n
    p = [[at.get("%s%d" % (k, i), A + (3 * i + j) * STEP) for i in range(n)] for j, k in enumerate(("x", "dy", "dw"))]
    return api.lib().jz_conv2d_bwd_weight_set(n, descs, arr(*p[0]), arr(*p[1]), arr(*p[2]), at.get("ws", A + 60 * STEP) if ws_bytes else None,
                                              ws_bytes, None)


def test_workspace_of_a_lone_member():
    assert call([FAST, STEM], 0) == api.JZ_ERR_WORKSPACE       # no room for the stem's padded copy
    assert call([STEM, FAST], 4096) == api.JZ_ERR_WORKSPACE


@pytest.mark.parametrize("layers", [[FAST, ODD], [ODD, FAST], [ODD, ODD], [FAST, FAST], [STEM, FAST, ODD]])
def test_overlaps_between_members(layers):
    last = len(layers) - 1
    at = lambda i, j: A + (3 * i + j) * STEP
    assert call(layers, **{"dw0": at(last, 2)}) == api.JZ_ERR_ALIAS                # two results
    for j, k in enumerate(("x", "dy")):
        assert call(layers, **{"dw0": at(last, j)}) == api.JZ_ERR_ALIAS            # a result and another member's operand
        assert call(layers, **{"dw%d" % last: at(0, j)}) == api.JZ_ERR_ALIAS


@pytest.mark.parametrize("layers", [[FAST, STEM], [STEM, ODD], [STEM, FAST, ODD]])
def test_workspace_over_another_member(layers):
    for i in range(len(layers)):
        for j in range(3):                                     # the stem's copy is 160 KB and more
            assert call(layers, ws=A + (3 * i + j) * STEP) == api.JZ_ERR_ALIAS


class _Tensor:                                                 # what binding looks at
    is_cuda, dtype = True, torch.float16
    is_contiguous = lambda self: True
    data_ptr = lambda self: A

    def __init__(self, n):
        self.numel = lambda: n


def test_bound_call_keeps_the_tensors_of_lists_that_change():
    d = api.conv_desc(*FAST)
    x, dy, dw = ([_Tensor(n)] for n in (d.N * d.H * d.W * d.C, d.N * d.P * d.Q * d.K, d.K * d.R * d.S * d.C))
    refs = [weakref.ref(t[0]) for t in (x, dy, dw)]
    bound = api.bind_conv2d_bwd_weight_set([d], x, dy, dw)
    for t in (x, dy, dw):
        t.clear()
    assert all(r() is not None for r in refs)                  # the call has their addresses
    del bound
    assert all(r() is None for r in refs)
