"""Operators that share the scratch memory of a stream: the results of their own, from any thread."""
import threading

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _shear(tsk, N, prec=0, steps=200, stream=None):
    y = 2 * np.pi * np.arange(N) / N
    op = tsk.create_kolmo2d(N, prec, stream=stream)
    tsk.set_params_kolmo(op, 20.0, 0.5, 0.005, steps * 0.005)
    tsk.set_base_parallel(op, 0.7 * np.sin(y) + 0.3 * np.sin(2 * y + 0.6), 0.7 * np.sin(y) + 1.2 * np.sin(2 * y + 0.6))
    x = op.new_state()
    x.copy_(torch.from_numpy(W.normal_real((x.numel(),), N + steps)))
    return op, x, op.new_state()


def _cgle(tsk, n, steps, stream=None):
    op = tsk.create_cgle1d(n, 30.0, stream=stream)
    tsk.set_params_cgle(op, 2.0, 0.2, -1.0, 0.38, -0.01, 0.01, 0.01 * steps)
    x = torch.from_numpy(W.cgle_start(n, 3)).cuda()
    return op, x, torch.zeros_like(x)


def test_second_operator_of_a_stream_allocates_no_second_workspace(tsk):
    # four matrices of 96 x 96 for each of 42 columns: 25 MB, once
    torch.cuda.synchronize()
    ops, free = [], []
    for _ in range(4):
        ops.append(_shear(tsk, 128))
        tsk.apply(*ops[-1])
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    assert free[0] - free[3] < 20 << 20
    for op, x, y in ops[1:]:
        assert torch.equal(y, ops[0][2])


def test_a_profile_set_again_is_the_one_that_is_squared(tsk):
    op, x, y = _shear(tsk, 48)
    tsk.apply(op, x, y)
    g = 2 * np.pi * np.arange(48) / 48
    tsk.set_base_parallel(op, 0.2 * np.sin(g) + 0.5 * np.sin(3 * g), 0.2 * np.sin(g) + 4.5 * np.sin(3 * g))
    z, st = op.new_state(), op.new_state()
    tsk.apply(op, x, z)
    tsk.set_tuning(op, 1)
    tsk.apply(op, x, st)
    assert not torch.equal(z, st) and torch.max(torch.abs(z - st)).item() <= 1e-11 * torch.max(torch.abs(st)).item()
    assert torch.max(torch.abs(z - y)).item() > 1e-3 * torch.max(torch.abs(y)).item()


def test_threads_with_operators_on_one_stream(tsk):
    # different sizes, precisions and kinds take turns in one memory; every result is that of a run alone
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ops = [_shear(tsk, 96), _shear(tsk, 64, 1), _cgle(tsk, 100, 900), _shear(tsk, 128, 0, 100), _cgle(tsk, 250, 1301)]
        want = []
        for op, x, y in ops:
            tsk.apply(op, x, y)
            want.append(y.clone())
            y.zero_()
    s.synchronize()
    errors = []

    def work(op, x, y, w):
        with torch.cuda.stream(s):
            for _ in range(30):
                tsk.apply(op, x, y)
                if not torch.equal(y, w):
                    errors.append(op)

    ts = [threading.Thread(target=work, args=(*o, w)) for o, w in zip(ops, want)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors


@pytest.mark.parametrize("late", [False, True])
def test_first_squared_call_while_another_stream_captures(tsk, late):
    # the memory, and the transform of a profile that was set before the parameters (late), come legally
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s1):
        cop = tsk.create_kolmo2d(64, 0)
        tsk.set_params_kolmo(cop, 20.0, 0.5, 0.005, 1.0)
        tsk.set_base_kolmogorov(cop, 4)
        cx, cy, cz = cop.new_state(), cop.new_state(), cop.new_state()
        cx.copy_(torch.from_numpy(W.normal_real((cx.numel(),), 1)))
        tsk.apply(cop, cx, cy)
    with torch.cuda.stream(s2):
        ref = _shear(tsk, 96)
        y = 2 * np.pi * np.arange(96) / 96
        op = tsk.create_kolmo2d(96, 0)
        if not late:
            tsk.set_params_kolmo(op, 20.0, 0.5, 0.005, 1.0)
        tsk.set_base_parallel(op, 0.7 * np.sin(y) + 0.3 * np.sin(2 * y + 0.6), 0.7 * np.sin(y) + 1.2 * np.sin(2 * y + 0.6))
        if late:
            tsk.set_params_kolmo(op, 20.0, 0.5, 0.005, 1.0)
        out = op.new_state()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s1):
        tsk.apply(cop, cx, cz)
        tsk.apply(op, ref[1], out)
    torch.cuda.synchronize()
    for _ in range(3):
        cz.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(cy, cz)
    tsk.apply(*ref)
    torch.cuda.synchronize()
    assert torch.equal(out, ref[2])
