"""Ginzburg-Landau integrations at the edges of their two forms: reduction levels left
out or kept, level pairs, and the dense propagator by squaring, against plain
64-bit references."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.cgle import CGLE
from oracle.optimal import cgle_apply_adjoint

pytestmark = pytest.mark.gpu
P = dict(U=2.0, c_u=0.2, c_d=-1.0, mu0=0.38, mu2=-0.01)


def _ref(n, hw, steps, dt):
    return CGLE(n=n, half_width=hw, dt=dt, T=steps * dt, **P)


def _op(tsk, n, hw, steps, dt):
    op = tsk.create_cgle1d(n, hw)
    tsk.set_params_cgle(op, P["U"], P["c_u"], P["c_d"], P["mu0"], P["mu2"], dt, steps * dt)
    return op


# (n, half width, steps, dt): dt and spacing set the number of levels that matter, from one (n = 2) over odd
# and even counts to all (dt = 0.5: strongly coupled); 300 steps of 513 nodes and 64 of 600 step with 1024
# threads; the last four square (one and several tiles, a remainder row, step counts with and without low bits).
# Bar: the stepper's 1e-12 of max |M u|, as for the other matvecs.
CASES = [(2, 1.0, 7, 0.01), (3, 1.0, 5, 0.5), (17, 3.0, 40, 0.01), (64, 50.0, 33, 0.01), (65, 10.0, 20, 0.02),
         (256, 50.0, 100, 0.01), (300, 20.0, 30, 0.5), (512, 30.0, 20, 0.01), (513, 50.0, 30, 0.01),
         (600, 20.0, 64, 0.01), (1024, 50.0, 10, 0.01),
         (16, 20.0, 600, 0.01), (33, 30.0, 1023, 0.01), (100, 50.0, 1024, 0.01), (250, 40.0, 1301, 0.01)]


@pytest.mark.parametrize("n,hw,steps,dt", CASES)
def test_propagator_and_adjoint_match_oracle(tsk, n, hw, steps, dt):
    print(f"cgle n={n} hw={hw} steps={steps} dt={dt}", flush=True)
    ref, op = _ref(n, hw, steps, dt), _op(tsk, n, hw, steps, dt)
    u = W.cgle_start(n, 5)
    x = torch.from_numpy(u).cuda()
    for apply, want in ((tsk.apply, ref.apply(u)), (tsk.apply_adjoint, cgle_apply_adjoint(ref, u))):
        y = torch.zeros_like(x)
        apply(op, x, y)
        assert np.max(np.abs(y.cpu().numpy() - want)) <= 1e-12 * np.max(np.abs(want))


@pytest.mark.parametrize("n,hw,omega,steps", [(16, 20.0, 0.7, 900), (48, 30.0, -0.55, 2047), (130, 40.0, -0.2, 1500)])
def test_squared_resolvent_matches_stepping_in_plain_arithmetic(tsk, n, hw, omega, steps):
    # Crank-Nicolson from rest with the trapezoidal forcing, as u(t) e^{-i omega t}.  Bar: 1e-11 of max |u|
    # (the resolvent tests' bar at small n is 1e-12 over 9000 steps of a shorter transient growth)
    print(f"cgle resolvent n={n} omega={omega} steps={steps}", flush=True)
    dt = 0.01
    ref, op = _ref(n, hw, 1, dt), _op(tsk, n, hw, 1, dt)
    tsk.set_resolvent(op, omega, steps * dt)
    f = W.cgle_start(n, 6)
    A = ref.matrix()
    I = np.eye(n)
    for adj in (False, True):
        L, w = (A.conj().T, -omega) if adj else (A, omega)
        lhs = np.linalg.inv(I - 0.5 * dt * L)
        B = lhs @ (I + 0.5 * dt * L)
        u = np.zeros(n, complex)
        c1 = lhs @ (0.5 * dt * (1 + np.exp(1j * w * dt)) * f)
        for s in range(steps):
            u = B @ u + np.exp(1j * w * dt * s) * c1
        want = u * np.exp(-1j * w * dt * steps)
        x = torch.from_numpy(f).cuda()
        y = torch.zeros_like(x)
        (tsk.apply_adjoint if adj else tsk.apply)(op, x, y)
        assert np.max(np.abs(y.cpu().numpy() - want)) <= 1e-11 * np.max(np.abs(want))


def test_batch_of_squaring_and_stepping_members_equals_single_runs_bitwise(tsk):
    # one node count, step counts of both forms and two squared groups
    ops, v0s = [], []
    for i, steps in enumerate((20, 1200, 700, 1200)):
        op = _op(tsk, 60, 30.0 + i, steps, 0.01)
        ops.append(op)
        v0s.append(torch.from_numpy(W.cgle_start(60, i)).cuda())
    rb = tsk.batch_arnoldi(ops, 10, 2, 0.0, v0s=v0s, want_vectors=True)
    for op, v0, b in zip(ops, v0s, rb):
        r = tsk.arnoldi(op, 10, 2, 0.0, v0=v0, want_vectors=True)
        assert np.array_equal(b["lam"], r["lam"]) and torch.equal(b["X"], r["X"])


def test_capture_of_a_first_squared_matvec_steps_instead(tsk):
    # no workspace can be allocated on a capturing stream: the captured matvec steps, and replays agree with the
    # squared one to rounding
    op_stream = torch.cuda.Stream()
    with torch.cuda.stream(op_stream):
        op = _op(tsk, 40, 30.0, 800, 0.01)
        x = torch.from_numpy(W.cgle_start(40, 3)).cuda()
        y = torch.zeros_like(x)
        z = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=op_stream):
        tsk.apply(op, x, y)
    g.replay()
    torch.cuda.synchronize()
    tsk.apply(op, x, z)
    torch.cuda.synchronize()
    assert torch.max(torch.abs(y - z)).item() <= 1e-12 * torch.max(torch.abs(z)).item()
    y.zero_()
    g.replay()
    torch.cuda.synchronize()
    assert torch.max(torch.abs(y - z)).item() <= 1e-12 * torch.max(torch.abs(z)).item()
