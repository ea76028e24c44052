"""Plans looked up by several threads at once (host logic only): each thread keeps its own table, more layers than it holds,
while another thread changes the tuning state; every answer is the one a single thread gets."""
import threading

import pytest


@pytest.fixture(scope="module")
def jz():
    from paper_1807_11205_amd import api
    api.lib()
    return api


def test_plans_of_concurrent_threads(jz):
    layers = [jz.conv_desc(n, h, h, c, k, r, r, s, r // 2) for n in (1, 3, 64) for h in (14, 29) for c, k in ((3, 64), (40, 24), (64, 128), (256, 30))
              for r, s in ((1, 1), (1, 2), (3, 1), (3, 2), (5, 3))]
    other = jz.conv_desc(17, 17, 17, 64, 64, 3, 3, 1, 1)       # the layer whose tuning changes: nobody asks for it
    ops = (jz.JZ_FWD, jz.JZ_BWD_DATA, jz.JZ_BWD_WEIGHT)
    ask = lambda d, op: (jz.jz_conv2d_workspace_bytes(op, d), jz.jz_conv2d_describe_plan(op, d), jz.jz_conv2d_f32_workspace_bytes(op, d))
    want = [ask(d, op) for d in layers for op in ops]
    assert len(want) > 256
    wrong, done = [], threading.Event()

    def reader(step):
        n = len(layers) * len(ops)
        for i in range(3 * n):
            j = i * step % n
            got = ask(layers[j // 3], ops[j % 3])
            if got != want[j]:
                wrong.append((j, got, want[j]))

    def tuner():
        while not done.is_set():
            jz.jz_conv2d_tune_set(jz.JZ_FWD, other, 64, 64, 32, 4, 4, 1)
            jz.jz_conv2d_tune_clear()

    threads = [threading.Thread(target=reader, args=(s,)) for s in (1, 7, 11, 1)]     # coprime to the number of plans
    t = threading.Thread(target=tuner)
    t.start()
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    done.set()
    t.join()
    assert not wrong, wrong[0]
