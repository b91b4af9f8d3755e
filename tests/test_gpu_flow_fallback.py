"""Two-dimensional integrations whose one-launch form cannot run: the integration behind a launch
that gave up, at the larger grids and for the nonlinear equation, and the stage launches that
follow it."""
import ctypes as C

import numpy as np
import pytest
import torch

import workloads as W
from oracle.fixedpoint import NonlinearKolmogorov
from oracle.kolmogorov import Kolmogorov, base_from_streamfunction
from oracle.optimal import kolmo_apply_adjoint

pytestmark = pytest.mark.gpu

DT = 0.005
DEFAULT, NONE, NONE_NOTED = -1, 0, -2


def _setup(tsk, N, prec, steps):
    U, V, Ox, Oy = base_from_streamfunction(W.random_base_modes(2, 1), N, 0.5)
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, 20.0, 0.5, DT, steps * DT)
    tsk.set_base_flow(op, U, V, Ox, Oy)
    ex = W.random_forcing_field(N, 0.5, 2, 7, 0.05)
    tsk.set_nonlinear(op, 4, 0.7, ex)
    ref = Kolmogorov(N, 0.5, 20.0, DT, steps * DT, U, V, Ox, Oy)
    nref = NonlinearKolmogorov(N, 0.5, 20.0, DT, steps * DT, U0=0.7, extra_forcing=ex)
    w = ref.project(W.kolmo_start_physical(N, 5))
    v = nref.omega_lam + nref.lin.project(W.random_forcing_field(N, 0.5, 3, 11, 0.2))
    return op, [(lambda x, y: tsk.apply(op, x, y), w, ref.apply(w)),
                (lambda x, y: tsk.apply_adjoint(op, x, y), w, kolmo_apply_adjoint(ref, w)),
                (lambda x, y: tsk.nonlinear_step(op, x, y, steps), v, nref.apply(v))]


def _state(tsk, op, w):
    x = op.new_state()
    tsk.from_physical(op, torch.from_numpy(np.ascontiguousarray(w)).to("cuda", op.state_dtype).reshape(-1), x)
    return x


def _close(tsk, op, y, want, prec):
    got = torch.zeros(op.N * op.N, dtype=op.state_dtype, device="cuda")
    tsk.to_physical(op, y, got)
    tol = 1e-11 if prec == 0 else 2e-5  # the pipeline's bars
    assert np.max(np.abs(got.double().cpu().numpy().reshape(op.N, op.N) - want)) <= tol * np.max(np.abs(want))


def _polls(tsk, op, n):
    assert tsk.load().tskx_flow_polls(op.h, n) == 0


def _gave_up(tsk, op):
    torch.cuda.synchronize()
    yes = C.c_int(-1)
    assert tsk.load().tskx_flow_gave_up(op.h, C.byref(yes)) == 0
    return yes.value


@pytest.mark.parametrize("N,steps,prec", [(32, 5, 0), (96, 2, 0), (128, 2, 1), (192, 1, 0), (256, 1, 0), (256, 1, 1)])
def test_integration_behind_a_launch_that_gave_up(tsk, N, steps, prec):
    print(f"flow repair N={N} steps={steps} prec={prec}", flush=True)
    op, calls = _setup(tsk, N, prec, steps)
    for run, w, want in calls:
        x, y, z = _state(tsk, op, w), op.new_state(), op.new_state()
        run(x, y)
        _polls(tsk, op, NONE)
        run(x, z)
        _close(tsk, op, z, want, prec)
        assert not torch.equal(y, z)  # the other transforms' rounding: it did give up
        assert _gave_up(tsk, op) == 0  # a forced one is not noted
        _polls(tsk, op, DEFAULT)
        run(x, z)
        assert torch.equal(y, z)


@pytest.mark.parametrize("N,steps,prec", [(16, 9, 1), (64, 3, 0), (96, 2, 1), (128, 2, 0), (256, 1, 1)])
def test_later_integrations_run_stage_by_stage(tsk, N, steps, prec):
    print(f"flow stages N={N} steps={steps} prec={prec}", flush=True)
    op, calls = _setup(tsk, N, prec, steps)
    for run, w, want in calls:
        x, y, z, s = _state(tsk, op, w), op.new_state(), op.new_state(), op.new_state()
        assert _gave_up(tsk, op) == 0
        run(x, y)
        _polls(tsk, op, NONE_NOTED)
        run(x, z)  # gives up and is repaired
        assert _gave_up(tsk, op) == 1
        _close(tsk, op, z, want, prec)
        run(x, s)  # does not try again
        _close(tsk, op, s, want, prec)
        assert not torch.equal(y, s)
        _polls(tsk, op, DEFAULT)
        run(x, z)
        assert torch.equal(y, z) and _gave_up(tsk, op) == 0
