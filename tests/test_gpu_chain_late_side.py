"""Weight gradients that arrive late: with the side streams held up in front of the backward pass, everything that reads a
gradient on the main stream (the sums of squares for the update's rates, the update) still has to see this step's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_side,proj", [(1, False), (2, False), (1, True)])
def test_an_update_waits_for_the_side_streams(n_side, proj):
    from paper_1807_11205_amd import resnet50
    out = []
    for sides in (None, [torch.cuda.Stream() for _ in range(n_side)]):
        net = resnet50.ResNet50Chain(batch=2, image=32, initial_loss_scale=512.0, hparams=dict(lr=1.0), proj_side=proj)
        for _ in range(2):
            net.forward(side=sides)
            for s in sides or []:
                with torch.cuda.stream(s):
                    torch.cuda._sleep(20_000_000)      # 10 ms or more; the backward pass takes about 2
            net.backward(side=sides)
            net.update()
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (net.grad, net.master, net.momentum)])
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))


def test_a_first_step_on_another_stream_than_the_current_one():
    """The side streams' workspaces are made by the first step that uses them: a current stream that is behind must not write
    to them while that step runs elsewhere."""
    from paper_1807_11205_amd import resnet50
    out = []
    for late in (False, True):
        net = resnet50.ResNet50Chain(batch=2, image=32, initial_loss_scale=512.0, hparams=dict(lr=1.0))
        main, sides = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(2)]
        torch.cuda.synchronize()
        if late:
            torch.cuda._sleep(20_000_000)
        net.step(main, sides if late else None)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (net.grad, net.master, net.momentum)])
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
