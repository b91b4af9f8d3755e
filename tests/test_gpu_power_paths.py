"""One-harmonic integrations with the path asserted: squared on the squaring side of the rule at
every tile count, in both directions and precisions; stepped below it in every launch shape."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.kolmogorov import Kolmogorov
from oracle.optimal import kolmo_apply_adjoint

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


# chains of 11 (one tile), 22 (two), 29 of an odd count (two), 43 (three), 64 (four), 69 (five), 85 and 86 modes
# (six); counts at and just above the line, and odd ones.  Bars: the stepper's, of max |M w|.
@pytest.mark.parametrize("N,nh,steps,prec,shift,adj", [
    (64, 4, 31, 0, 0.2, False), (64, 4, 33, 0, 0.0, True), (128, 4, 33, 0, 0.0, False), (128, 3, 47, 0, 0.7, True),
    (256, 4, 81, 0, 0.0, False), (256, 4, 83, 0, 0.1, True), (384, 4, 185, 0, 0.3, False), (384, 4, 193, 0, 0.0, True),
    (512, 5, 147, 0, 0.0, False), (512, 5, 161, 0, 0.2, True), (128, 1, 151, 0, 0.2, False), (512, 4, 165, 0, 0.0, True),
    (64, 4, 33, 1, 0.0, False), (64, 4, 35, 1, 0.2, True), (128, 4, 37, 1, 0.0, False), (128, 4, 51, 1, 0.1, True),
    (256, 4, 65, 1, 0.4, False), (256, 4, 77, 1, 0.0, True), (384, 4, 321, 1, 0.0, False), (384, 4, 325, 1, 0.2, True),
    (512, 5, 81, 1, 0.0, False), (512, 5, 83, 1, 0.1, True), (512, 4, 85, 1, 0.0, False), (512, 4, 93, 1, 0.0, True)])
def test_squared_path_matches_oracle_and_is_taken(tsk, N, nh, steps, prec, shift, adj):
    print(f"power path N={N} nh={nh} steps={steps} prec={prec} adj={adj}", flush=True)
    op, U = _op(tsk, N, nh, steps, prec, shift)
    Ug = np.repeat(U[:, None], N, axis=1)
    zero = np.zeros_like(Ug)
    ref = Kolmogorov(N, 0.5, 20.0, DT, steps * DT, Ug, zero, zero, nh * nh * Ug)
    w = ref.project(W.kolmo_start_physical(N, 11))
    x, y, z = op.new_state(), op.new_state(), op.new_state()
    tsk.from_physical(op, torch.from_numpy(w).to("cuda", op.state_dtype).reshape(-1), x)
    apply = tsk.apply_adjoint if adj else tsk.apply
    apply(op, x, y)
    _step_only(tsk, op, True)
    apply(op, x, z)
    assert not torch.equal(y, z)
    want = kolmo_apply_adjoint(ref, w) if adj else ref.apply(w)
    tol = 1e-11 if prec == 0 else 2e-5
    for s in (y, z):
        got = torch.zeros(N * N, dtype=op.state_dtype, device="cuda")
        tsk.to_physical(op, s, got)
        assert np.max(np.abs(got.double().cpu().numpy().reshape(N, N) - want)) <= tol * np.max(np.abs(want))


@pytest.mark.parametrize("N,nh,steps,prec,adj", [
    (64, 4, 27, 0, False), (128, 4, 31, 0, False), (128, 4, 43, 0, True), (256, 4, 79, 0, False), (384, 4, 183, 0, False),
    (512, 4, 145, 0, False), (64, 4, 31, 1, False), (256, 4, 75, 1, True), (384, 4, 319, 1, False), (384, 4, 200, 1, True)])
def test_below_the_line_it_steps(tsk, N, nh, steps, prec, adj):
    op, _ = _op(tsk, N, nh, steps, prec)
    x, y, z = op.new_state(), op.new_state(), op.new_state()
    x.copy_(torch.from_numpy(W.normal_real((x.numel(),), 4)))
    apply = tsk.apply_adjoint if adj else tsk.apply
    apply(op, x, y)
    _step_only(tsk, op, True)
    apply(op, x, z)
    assert torch.equal(y, z)


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
