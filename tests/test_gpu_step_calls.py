"""How many library calls a recorded training step makes."""
import pytest
import torch

from paper_1908_00213_amd import steps, workloads as W

pytestmark = pytest.mark.gpu


def test_calls_of_a_small_classifiers_step():
    w = W.config1()
    tr = steps.MLPTrainer(w.params, w.batch, w.act, w.lr, lowp=False)
    x, t = torch.from_numpy(w.xs[0]).cuda(), torch.from_numpy(w.ts[0]).cuda()
    # 3 forward products, loss with its gradient, the backward of 3 layers, 1 update
    assert tr.n_calls(x, t) == 8
    # ... whose backward calls stand for 3 weight, 3 bias and 2 input gradients
    assert tr.n_launch_calls(x, t) == 13
