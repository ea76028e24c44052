"""Split counts of backward-weight (host logic only): alone a launch fills the chip, tune.share_chip restores the recorded
counts for steps that run it beside other streams, jz_conv2d_tune_clear takes them back."""
import re

import pytest


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    return api


def splits_and_workgroups(jz, d):
    m = re.search(r"(\d+) x (\d+) tiles, (\d+) splits", jz.jz_conv2d_describe_plan(jz.JZ_BWD_WEIGHT, d))
    tm, tn, sp = (int(v) for v in m.groups())
    return sp, tm * tn * sp


@pytest.mark.parametrize("H,C,K,R,recorded", [(28, 128, 512, 1, 12), (14, 256, 1024, 1, 3), (14, 256, 256, 3, 3), (56, 64, 64, 3, 64)])
def test_backward_weight_fills_the_chip_alone_and_shares_it_on_request(jz, H, C, K, R, recorded):
    from paper_1807_11205_amd import tune
    d = jz.conv_desc(64, H, H, C, K, R, R, 1, R // 2)
    alone, wgs = splits_and_workgroups(jz, d)
    assert alone > recorded and 160 <= wgs <= 1024
    other = jz.conv_desc(63, H, H, C, K, R, R, 1, R // 2)     # in no table
    assert 160 <= splits_and_workgroups(jz, other)[1] <= 1280
    try:
        assert tune.share_chip([d, other]) == 1
        assert splits_and_workgroups(jz, d)[0] == recorded
    finally:
        jz.jz_conv2d_tune_clear()
    assert splits_and_workgroups(jz, d)[0] == alone
