"""Integration about profiles of several harmonics by repeated squaring of the
column matrices (colmatrix.hpp) against the oracle's transform stepper, at the column
lengths and bandwidths where its tiles change."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.kolmogorov import Kolmogorov
from oracle.optimal import kolmo_apply_adjoint

pytestmark = pytest.mark.gpu

DT = 0.005


def _op(tsk, N, prec, steps, harmonics):
    y = 2 * np.pi * np.arange(N) / N
    U = sum(a * np.sin(h * y + 0.3 * h) for h, a in harmonics)
    d = sum(a * h * h * np.sin(h * y + 0.3 * h) for h, a in harmonics)
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, 20.0, 0.5, DT, steps * DT)
    tsk.set_base_parallel(op, U, d)
    z = np.zeros((N, N))
    ref = Kolmogorov(N, 0.5, 20.0, DT, steps * DT, np.repeat(U[:, None], N, 1), z, z, np.repeat(d[:, None], N, 1))
    return op, ref


# modes per column: 11 (16), 21 (32), 43 (64, a remainder in the third tile), 63 (96), 85 (128), 127 (192, two
# tiles per wavefront from here), 171 (256), 255 (384).  Harmonics 1 + 2: a narrow band; 4 + 8 + 12: a period-4
# profile; up to N / 3 + 1: products that wrap on the grid.  Step counts: the smallest that squares, powers of two
# and neighbours.  Bars: those of the stepper, 1e-11 (FP64) and 2e-5 (FP32) of max |M w|.
NARROW, PERIOD = ((1, 0.7), (2, 0.3)), ((4, 0.6), (8, 0.3), (12, 0.1))


def _wide(N):
    return ((1, 0.6), (N // 5, 0.02), (N // 3 + 1, 0.002))


@pytest.mark.parametrize("N,steps,prec,base,adj", [
    (16, 16, 0, "wide", False), (16, 33, 0, "narrow", True), (32, 31, 0, "wide", True),
    (48, 17, 0, "narrow", False),
    (64, 40, 0, "narrow", False), (96, 64, 0, "period", True), (96, 100, 0, "wide", False),
    (128, 63, 0, "narrow", False), (128, 64, 0, "wide", True), (192, 65, 0, "narrow", True),
    (192, 60, 0, "wide", False), (256, 160, 0, "narrow", False), (384, 200, 0, "period", False),
    (384, 300, 0, "wide", True), (16, 16, 1, "narrow", False), (64, 33, 1, "wide", True),
    (96, 47, 1, "narrow", False), (192, 50, 1, "wide", False), (256, 128, 1, "narrow", True)])
def test_squared_columns_match_oracle(tsk, N, steps, prec, base, adj):
    print(f"columns N={N} steps={steps} prec={prec} base={base} adj={adj}", flush=True)
    op, ref = _op(tsk, N, prec, steps, {"narrow": NARROW, "period": PERIOD, "wide": _wide(N)}[base])
    w = ref.project(W.kolmo_start_physical(N, 11))
    x, out = op.new_state(), op.new_state()
    tsk.from_physical(op, torch.from_numpy(w).to("cuda", op.state_dtype).reshape(-1), x)
    apply = tsk.apply_adjoint if adj else tsk.apply
    apply(op, x, out)
    stepped = op.new_state()
    tsk.set_tuning(op, 1)
    apply(op, x, stepped)
    # squared (the rounding of the 384^2 period-4 samples fills the band, which puts 200 steps at the break-even)
    assert (N, steps) == (384, 200) or not torch.equal(out, stepped)
    got = torch.zeros(N * N, dtype=op.state_dtype, device="cuda")
    tsk.to_physical(op, out, got)
    want = kolmo_apply_adjoint(ref, w) if adj else ref.apply(w)
    tol = 1e-11 if prec == 0 else 2e-5
    assert np.max(np.abs(got.double().cpu().numpy().reshape(N, N) - want)) <= tol * np.max(np.abs(want))


def test_captured_matvec_steps_and_a_forced_variant_steps(tsk):
    # a graph must not share the operator's workspace: the captured matvec is the stepper's, bit for bit
    # (of one column per wavefront, without the launches that time the variants)
    N, s = 64, torch.cuda.Stream()
    with torch.cuda.stream(s):
        op, _ = _op(tsk, N, 0, 40, NARROW)
        x, sq, st, cp = (op.new_state() for _ in range(4))
        tsk.from_physical(op, torch.from_numpy(W.kolmo_start_physical(N, 3)).cuda().reshape(-1), x)
        tsk.apply(op, x, sq)
        tsk.set_tuning(op, 1)
        tsk.apply(op, x, st)
        tsk.set_tuning(op, 0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        tsk.apply(op, x, cp)
    for _ in range(2):
        cp.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(cp, st) and not torch.equal(sq, st)
        assert torch.max(torch.abs(sq - st)).item() <= 1e-12 * torch.max(torch.abs(st)).item()
