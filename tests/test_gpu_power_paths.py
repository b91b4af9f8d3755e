"""One-harmonic integrations with the path asserted: squared on the squaring side of the rule at
every tile count, in both directions and precisions; stepped below it in every launch shape."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

DT = 0.005


def _op(tsk, N, nh, steps, prec, shift=0.0, Re=20.0):
    y = 2 * np.pi * np.arange(N) / N
    U = 0.8 * np.sin(nh * (y - shift))
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, Re, 0.5, DT, steps * DT)
    tsk.set_base_parallel(op, U, nh * nh * U)
    assert tsk.get_tuning(op) == -2
    return op, U


def _step_only(tsk, op, on):
    assert tsk.load().tskx_step_only(op.h, int(on)) == 0


@pytest.mark.parametrize("prec", [0, 1])
def test_stepping_launch_shapes_agree_bitwise(tsk, prec):
    # 1, 2 and 4 wavefronts per workgroup of the stepper, alone, transposed and in a batch
    ops, v0s = [], []
    for i, (N, nh) in enumerate(((64, 4), (128, 4), (384, 4), (512, 4))):
        op, _ = _op(tsk, N, nh, 200, prec, Re=12.0 + i)
        _step_only(tsk, op, True)
        x = op.new_state()
        x.copy_(torch.from_numpy(W.normal_real((x.numel(),), 5 + i)))
        x /= torch.linalg.norm(x)
        for apply in (tsk.apply, tsk.apply_adjoint):
            outs = []
            for w in (1, 2, 4, 0):
                tsk.set_stepper_waves(op, w)
                y = op.new_state()
                apply(op, x, y)
                assert tsk.get_stepper_waves(op) == w if w else tsk.get_stepper_waves(op) in (1, 2, 4)
                outs.append(y)
            assert all(torch.equal(outs[0], o) for o in outs[1:])
        ops.append(op)
        v0s.append(x)
    res = []
    for w in (1, 2, 4):
        for op in ops:
            tsk.set_stepper_waves(op, w)
        res.append(tsk.batch_arnoldi(ops, 12, 2, 0.0, v0s=v0s))
    for op, v0, a, b, c in zip(ops, v0s, *res):
        assert np.array_equal(a["lam"], b["lam"]) and np.array_equal(a["lam"], c["lam"])
        assert np.array_equal(a["lam"], tsk.arnoldi(op, 12, 2, 0.0, v0=v0)["lam"])


def test_squared_matvec_steers_no_later_stepper(tsk):
    # the shape of the last forward launch that stepped stays; a squared one reports its own
    op, _ = _op(tsk, 128, 4, 200, 0)
    x, y = op.new_state(), op.new_state()
    x.copy_(torch.from_numpy(W.normal_real((x.numel(),), 6)))
    assert tsk.get_stepper_waves(op) == 0
    _step_only(tsk, op, True)
    tsk.apply(op, x, y)
    stepped = tsk.get_stepper_waves(op)
    _step_only(tsk, op, False)
    tsk.apply(op, x, y)
    assert tsk.get_stepper_waves(op) == 4
    _step_only(tsk, op, True)
    tsk.apply(op, x, y)
    assert tsk.get_stepper_waves(op) == stepped
