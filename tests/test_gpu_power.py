"""Integration of one-harmonic base flows by repeated squaring (colpower.hpp) against
the oracle's full transform stepper, at the chain lengths where its tiles change."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.kolmogorov import Kolmogorov
from oracle.optimal import kolmo_apply_adjoint

pytestmark = pytest.mark.gpu

DT = 0.005


# chains per column nh and their longest length: 96/4: 16 (one full tile), 64/2: 22, 128/5: 17
# (one mode beyond a tile), 192/4: 32 (two full tiles), 128/3: 29 (odd nh: no chain is its own
# mirror image but c = 0), 256/4: 43, 384/4: 64, 256/2: 86, 128/1: 85 (a single chain), 512/4: 86.
# Step counts: near the smallest that square (both sides of the rule), powers of two and their neighbours.
# Bars: those of the stepper, 1e-11 (FP64) and 2e-5 (FP32) of max |M w|.
@pytest.mark.parametrize("N,nh,steps,prec,shift,adj", [
    (16, 4, 16, 0, 0.0, False), (96, 4, 31, 0, 0.0, False), (64, 2, 64, 0, 0.3, False), (128, 5, 33, 0, 0.0, True),
    (192, 4, 127, 0, 0.0, False), (128, 3, 100, 0, 0.7, True), (256, 4, 128, 0, 0.0, False),
    (384, 4, 177, 0, 0.1, True), (256, 2, 120, 0, 0.0, False), (128, 1, 121, 0, 0.2, False),
    (512, 4, 120, 0, 0.0, True), (96, 4, 17, 1, 0.2, True), (128, 4, 200, 1, 0.0, False),
    (256, 4, 57, 1, 0.4, False), (384, 4, 137, 1, 0.0, False), (512, 4, 81, 1, 0.0, False)])
def test_squaring_matches_oracle(tsk, N, nh, steps, prec, shift, adj):
    print(f"power N={N} nh={nh} steps={steps} prec={prec} shift={shift} adj={adj}", flush=True)
    y = 2 * np.pi * np.arange(N) / N
    U = 0.8 * np.sin(nh * (y - shift))
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, 20.0, 0.5, DT, steps * DT)
    tsk.set_base_parallel(op, U, nh * nh * U)
    assert tsk.get_tuning(op) == -2
    Ug = np.repeat(U[:, None], N, axis=1)
    zero = np.zeros_like(Ug)
    ref = Kolmogorov(N, 0.5, 20.0, DT, steps * DT, Ug, zero, zero, nh * nh * Ug)
    w = ref.project(W.kolmo_start_physical(N, 11))
    x, out = op.new_state(), op.new_state()
    tsk.from_physical(op, torch.from_numpy(w).to("cuda", op.state_dtype).reshape(-1), x)
    (tsk.apply_adjoint if adj else tsk.apply)(op, x, out)
    got = torch.zeros(N * N, dtype=op.state_dtype, device="cuda")
    tsk.to_physical(op, out, got)
    want = kolmo_apply_adjoint(ref, w) if adj else ref.apply(w)
    tol = 1e-11 if prec == 0 else 2e-5
    assert np.max(np.abs(got.double().cpu().numpy().reshape(N, N) - want)) <= tol * np.max(np.abs(want))


def test_batch_that_squares_and_steps_equals_single_runs_bitwise(tsk):
    # 48^2 and 128^2 square, 64^2 with 12 steps and 384^2 with 100 steps step: two launches, one group
    cfg = [(48, 200), (64, 12), (128, 100), (384, 100), (256, 200)]
    ops, v0s = [], []
    for i, (N, steps) in enumerate(cfg):
        op = tsk.create_kolmo2d(N, tsk.TSK_FP64)
        tsk.set_params_kolmo(op, 15.0 + i, 0.5, DT, steps * DT)
        tsk.set_base_kolmogorov(op, 4)
        x = op.new_state()
        tsk.from_physical(op, torch.from_numpy(W.kolmo_start_physical(N, i)).cuda().reshape(-1), x)
        ops.append(op)
        v0s.append(x)
    rb = tsk.batch_arnoldi(ops, 12, 2, 0.0, v0s=v0s, want_vectors=True)
    for op, v0, b in zip(ops, v0s, rb):
        r = tsk.arnoldi(op, 12, 2, 0.0, v0=v0, want_vectors=True)
        assert np.array_equal(b["lam"], r["lam"]) and np.array_equal(b["res"], r["res"])
        assert torch.equal(b["X"], r["X"])
