"""The two-dimensional pipeline in one launch (genflow.hpp): every grid it covers against the
oracle, several launches per call, launches side by side, graphs, and the way out when a
wait between workgroups gives up."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.fixedpoint import NonlinearKolmogorov
from oracle.kolmogorov import Kolmogorov, base_from_streamfunction
from oracle.optimal import kolmo_apply_adjoint

pytestmark = pytest.mark.gpu

DT = 0.005


def _flow(tsk, N, prec, steps, seed=1):
    U, V, Ox, Oy = base_from_streamfunction(W.random_base_modes(2, seed), N, 0.5)
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, 20.0, 0.5, DT, steps * DT)
    tsk.set_base_flow(op, U, V, Ox, Oy)
    return op, Kolmogorov(N, 0.5, 20.0, DT, steps * DT, U, V, Ox, Oy)


def _state(tsk, op, w):
    x = op.new_state()
    tsk.from_physical(op, torch.from_numpy(np.ascontiguousarray(w)).to("cuda", op.state_dtype).reshape(-1), x)
    return x


def _close(tsk, op, y, want, prec):
    got = torch.zeros(op.N * op.N, dtype=op.state_dtype, device="cuda")
    tsk.to_physical(op, y, got)
    tol = 1e-11 if prec == 0 else 2e-5  # the pipeline's bars
    assert np.max(np.abs(got.double().cpu().numpy().reshape(op.N, op.N) - want)) <= tol * np.max(np.abs(want))


# all grids of one launch (lanes without a point at 16 .. 48, two and three runs of kx at 192 and 256); 515 steps at
# 16 are two launches, 1025 three
@pytest.mark.parametrize("N,steps,prec", [(16, 515, 0), (16, 1025, 1), (32, 7, 0), (32, 1, 1), (48, 5, 1), (64, 3, 0),
                                          (64, 3, 1), (96, 2, 0), (96, 2, 1), (128, 1, 0), (192, 2, 0), (192, 2, 1),
                                          (256, 2, 0), (256, 2, 1)])
def test_forward_adjoint_and_nonlinear_match_oracle(tsk, N, steps, prec):
    print(f"flow N={N} steps={steps} prec={prec}", flush=True)
    op, ref = _flow(tsk, N, prec, steps)
    w = ref.project(W.kolmo_start_physical(N, 5))
    x, y = _state(tsk, op, w), op.new_state()
    tsk.apply(op, x, y)
    _close(tsk, op, y, ref.apply(w), prec)
    tsk.apply_adjoint(op, x, y)
    _close(tsk, op, y, kolmo_apply_adjoint(ref, w), prec)
    n = min(steps, 10)
    ex = W.random_forcing_field(N, 0.5, 2, 7, 0.05)
    tsk.set_nonlinear(op, 4, 0.7, ex)
    nref = NonlinearKolmogorov(N, 0.5, 20.0, DT, n * DT, U0=0.7, extra_forcing=ex)
    w = nref.omega_lam + nref.lin.project(W.random_forcing_field(N, 0.5, 3, 11, 0.2))
    tsk.nonlinear_step(op, _state(tsk, op, w), y, n)
    _close(tsk, op, y, nref.apply(w), prec)


@pytest.mark.parametrize("N,steps,prec", [(16, 600, 0), (48, 3, 1), (64, 2, 0)])
def test_waits_that_give_up_leave_the_right_result(tsk, N, steps, prec):
    # no poll is repeated: the launch gives up, and the integration behind it takes over; afterwards all is as before
    print(f"flow gives up N={N} steps={steps} prec={prec}", flush=True)
    op, ref = _flow(tsk, N, prec, steps)
    w = ref.project(W.kolmo_start_physical(N, 5))
    x, y, z = _state(tsk, op, w), op.new_state(), op.new_state()
    for apply, want in ((tsk.apply, ref.apply(w)), (tsk.apply_adjoint, kolmo_apply_adjoint(ref, w))):
        apply(op, x, y)
        assert tsk.load().tskx_flow_polls(op.h, 0) == 0
        apply(op, x, z)
        _close(tsk, op, z, want, prec)
        assert not torch.equal(y, z)  # the other transforms' rounding: it did give up
        assert tsk.load().tskx_flow_polls(op.h, -1) == 0
        apply(op, x, z)
        assert torch.equal(y, z)


def test_launches_on_four_streams_agree_with_one_after_the_other(tsk):
    runs = []
    for i in range(4):
        with torch.cuda.stream(torch.cuda.Stream()):
            op, ref = _flow(tsk, 256, 0, 20, seed=i)
            x = _state(tsk, op, W.kolmo_start_physical(256, i))
            runs.append((op, x, op.new_state(), op.new_state()))
    torch.cuda.synchronize()
    for op, x, y, _ in runs:
        tsk.apply(op, x, y)
        torch.cuda.synchronize()
    for op, x, _, z in runs:
        tsk.apply(op, x, z)
    torch.cuda.synchronize()
    for op, x, y, z in runs:
        assert torch.equal(y, z)


def test_graph_replays_between_eager_calls(tsk):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        op, ref = _flow(tsk, 64, 0, 4)
        x = _state(tsk, op, W.kolmo_start_physical(64, 3))
        y, z = op.new_state(), op.new_state()
        tsk.apply(op, x, y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        tsk.apply(op, x, z)
    for i in range(4):
        z.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, z)
        if i % 2:
            tsk.apply(op, y, z)
            torch.cuda.synchronize()
