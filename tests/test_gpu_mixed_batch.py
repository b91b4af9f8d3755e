"""Batches that mix base flows of both kinds: each instance gets the bits of its own run."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _ops(tsk):
    # profiles of two harmonics whose matvecs square, a one-harmonic base that squares, a two-dimensional base
    ops, v0s = [], []
    for i, (N, kind) in enumerate(((48, "shear"), (32, "flow2d"), (96, "shear"), (64, "sine"))):
        y = 2 * np.pi * np.arange(N) / N
        op = tsk.create_kolmo2d(N, tsk.TSK_FP64)
        tsk.set_params_kolmo(op, 15.0 + i, 0.5, 0.005, 0.5)
        if kind == "sine":
            tsk.set_base_kolmogorov(op, 4)
        elif kind == "shear":
            tsk.set_base_parallel(op, 0.7 * np.sin(y) + 0.3 * np.sin(2 * y + 0.6),
                                  0.7 * np.sin(y) + 1.2 * np.sin(2 * y + 0.6))
        else:
            X, Y = np.meshgrid(0.5 * y, y)
            a, b = np.sin(4 * Y), 0.2 * np.cos(2 * X + Y)
            tsk.set_base_flow(op, a, 0.1 * b, 0.1 * b, 16 * a)
        x = op.new_state()
        tsk.from_physical(op, torch.from_numpy(W.kolmo_start_physical(N, i)).cuda().reshape(-1), x)
        ops.append(op)
        v0s.append(x)
    return ops, v0s


def test_mixed_batch_equals_single_runs_bitwise(tsk):
    ops, v0s = _ops(tsk)
    rb = tsk.batch_arnoldi(ops, 12, 2, 0.0, v0s=v0s, want_vectors=True)
    for op, v0, b in zip(ops, v0s, rb):
        r = tsk.arnoldi(op, 12, 2, 0.0, v0=v0, want_vectors=True)
        assert np.array_equal(b["lam"], r["lam"]) and np.array_equal(b["res"], r["res"])
        assert torch.equal(b["X"], r["X"])


def test_mixed_batch_of_restarted_runs_equals_single_ones_bitwise(tsk):
    ops, v0s = _ops(tsk)
    rb = tsk.batch_krylov_schur(ops, 10, 2, 1e-12, delta=0.1, max_restarts=2, v0s=v0s, want_vectors=True)
    assert any(b["n_restarts"] > 0 for b in rb)
    for op, v0, b in zip(ops, v0s, rb):
        r = tsk.batch_krylov_schur([op], 10, 2, 1e-12, delta=0.1, max_restarts=2, v0s=[v0], want_vectors=True)[0]
        assert b["n_matvec"] == r["n_matvec"] and np.array_equal(b["lam"], r["lam"])
        assert torch.equal(b["X"], r["X"])
