"""Gradients where the launches of a training step change: products split or not, weight
gradients that need slabs of their own (narrow layers, large batches), tile and column
remainders."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mlp
from test_gpu_mlp import GRAD_TOL, _inputs, _net

pytestmark = pytest.mark.gpu


# (16, 600): W3's gradient is split; (272, 65): a column of tiles with one row, 64-column remainders in the bias
# sums; (512, 128): the output product in two slabs; (1024, 3): fewer rows than the unrolled sums
@pytest.mark.parametrize("width,B", [(16, 600), (272, 65), (512, 128), (1024, 3), (16, 1)])
def test_gradients_match_oracle_at_the_edges(tsk, width, B):
    net, P = _net(tsk, width, 11)
    raw = _inputs(B, 12)
    T = (0.1 * W.normal_real((B, mlp.OUT), 13)).astype(np.float32)
    g, loss = tsk.mlp_gradients(net, torch.from_numpy(raw).cuda(), torch.from_numpy(T).cuda())
    G = mlp.unflatten(g.cpu().numpy().astype(np.float64), width)
    Gr, loss_r = mlp.grads(P, mlp.features(raw.astype(np.float64)), T.astype(np.float64))
    assert abs(loss - loss_r) <= 1e-5 * loss_r
    for k in mlp.ORDER:
        assert np.linalg.norm(G[k] - Gr[k]) <= GRAD_TOL * np.linalg.norm(Gr[k]), k


def test_a_training_step_is_the_gradient_and_one_adam_step(tsk):
    # the fused step against the gradient call and Adam in FP32 arithmetic: first step, m = (1 - b1) g and
    # v = (1 - b2) g^2, so w moves by lr g / (|g| + eps) up to rounding
    width, B, lr = 48, 64, 1e-3
    net, P = _net(tsk, width, 3)
    x = torch.from_numpy(_inputs(B, 4)).cuda()
    t = torch.from_numpy((0.1 * W.normal_real((B, mlp.OUT), 5)).astype(np.float32)).cuda()
    w0 = tsk.mlp_get_params(net).astype(np.float64)
    g, loss = tsk.mlp_gradients(net, x, t)
    losses = tsk.mlp_train(net, x, t, 1, lr)
    assert losses[0] == loss
    g = g.cpu().numpy().astype(np.float64)
    step = tsk.mlp_get_params(net).astype(np.float64) - w0
    want = -lr * g / (np.abs(g) + 1e-8)
    assert np.max(np.abs(step - want)) <= 1e-5 * lr + 2.0 ** -24 * np.max(np.abs(w0))
