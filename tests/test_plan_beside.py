"""jz_conv2d_bwd_weight_beside's plans (host logic only): the split of a weight gradient that shares the chip belongs to the call,
not to the process."""
import ctypes
import re
import threading

import pytest

from test_plan_splits import jz, splits_and_workgroups  # noqa: F401


def beside(jz, d):  # noqa: F811
    from paper_1807_11205_amd import tune
    return tune.plan_choice(jz.jz_conv2d_describe_plan(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, d))


@pytest.mark.parametrize("H,C,K,R,recorded", [(28, 128, 512, 1, 12), (14, 256, 1024, 1, 3), (14, 256, 256, 3, 3), (56, 64, 64, 3, 64)])
def test_recorded_layers_keep_their_shared_split_and_nobody_elses_changes(jz, H, C, K, R, recorded):  # noqa: F811
    d = jz.conv_desc(64, H, H, C, K, R, R, 1, R // 2)
    alone = splits_and_workgroups(jz, d)
    assert beside(jz, d)[5] == recorded < alone[0]
    seen = []
    t = threading.Thread(target=lambda: seen.append(splits_and_workgroups(jz, d)))
    t.start()
    t.join()
    assert seen == [alone] and splits_and_workgroups(jz, d) == alone
    assert jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, d) < jz.jz_conv2d_workspace_bytes(jz.JZ_BWD_WEIGHT, d)


def test_other_layers_share_the_chip_too(jz):  # noqa: F811
    from paper_1807_11205_amd import shapes
    total = lambda op, n: sum(jz.jz_conv2d_workspace_bytes(op, jz.conv_desc(n, c.H, c.H, c.C, c.K, c.R, c.R, c.stride, c.pad))
                              for c in shapes.resnet50_convs() if c.C > 4)
    fewer = 0
    for c in shapes.resnet50_convs():
        d = jz.conv_desc(63, c.H, c.H, c.C, c.K, c.R, c.R, c.stride, c.pad)      # in no table
        if c.H <= 28:
            a, b = splits_and_workgroups(jz, d)[1], jz.jz_conv2d_describe_plan(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, d)
            tm, tn, sp = (int(v) for v in re.search(r"(\d+) x (\d+) tiles, (\d+) splits", b).groups())
            assert tm * tn * sp <= 256
            fewer += tm * tn * sp < a
    assert fewer >= 20 and total(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, 63) < total(jz.JZ_BWD_WEIGHT, 63)


def test_the_flag_belongs_to_the_weight_gradient(jz):  # noqa: F811
    n = ctypes.c_size_t(0)
    d = jz.conv_desc(64, 56, 56, 64, 64, 3, 3, 1, 1)
    for op in (jz.JZ_FWD, jz.JZ_BWD_DATA):
        assert jz.lib().jz_conv2d_workspace_bytes(op | jz.JZ_BESIDE, ctypes.byref(d), ctypes.byref(n)) == jz.JZ_ERR_UNSUPPORTED
    assert jz.lib().jz_conv2d_tune_set(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, ctypes.byref(d), 64, 64, 32, 4, 4, 1) == jz.JZ_ERR_UNSUPPORTED
    assert jz.lib().jz_gemm_fc(jz.JZ_BWD_WEIGHT | jz.JZ_BESIDE, 4, 8, 8, None, None, None, None, 0, None) == jz.JZ_ERR_UNSUPPORTED
    A = 0x10000000
    assert jz.lib().jz_conv2d_bwd_weight_beside(ctypes.byref(d), None, A, A + (1 << 20), None, 0, None, None) == jz.JZ_ERR_NULL
    assert jz.lib().jz_conv2d_bwd_weight_beside(ctypes.byref(d), A, A + (1 << 28), A + (1 << 29), None, 0, None, None) == jz.JZ_ERR_WORKSPACE
