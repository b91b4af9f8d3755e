"""Integrations by repeated squaring keep the damped modes: against the power of the
one-step matrix in extended precision, mode by mode."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

DT = 0.005
LD, CLD = np.longdouble, np.clongdouble


def _power(S, n):
    P = np.eye(len(S), dtype=S.dtype)
    for b in bin(n)[2:]:
        P = P @ P
        P = P @ S if b == "1" else P
    return P


def _majorant(S, x, n, parts=8):
    """max over splits q of |S^(n-q)| (|S^q| |x|): what one relative rounding of the state or of a power
    anywhere on the way can move the result by."""
    s = n // parts
    P = _power(S, s)
    powers = [_power(S, n - parts * s)]
    for _ in range(parts):
        powers.append(powers[-1] @ P)
    left = [np.eye(len(S), dtype=S.dtype)]
    for _ in range(parts):
        left.append(left[-1] @ P)
    return np.max([np.abs(left[parts - i]) @ (np.abs(powers[i]) @ np.abs(x)) for i in range(parts + 1)], axis=0)


def _lawson(A, K2, Re):
    """One-step matrix of the integrating-factor RK4 scheme, generator A, damping K2 / Re."""
    h = LD(DT)
    E = np.diag(np.exp(-K2 * h / (2 * LD(Re)))).astype(A.dtype)
    E1, I = E @ E, np.eye(len(A), dtype=A.dtype)
    k1 = A
    k2 = A @ (E @ (I + h / 2 * k1))
    k3 = A @ (E + h / 2 * k2)
    k4 = A @ (E1 + h * E @ k3)
    return E1 + h / 6 * (E1 @ k1 + 2 * E @ k2 + 2 * E @ k3 + k4)


def _op(tsk, N, Re, prec, steps):
    op = tsk.create_kolmo2d(N, prec)
    tsk.set_params_kolmo(op, Re, 0.5, DT, steps * DT)
    return op


def _run(tsk, op, seed, adj):
    x, y = op.new_state(), op.new_state()
    x.copy_(torch.from_numpy(W.normal_real((x.numel(),), seed)))
    (tsk.apply_adjoint if adj else tsk.apply)(op, x, y)
    return x.cpu().numpy(), y.cpu().numpy()


def _column(v, N, kx):
    M = (N - 1) // 3
    s = v[2 * M + (kx - 1) * 2 * (2 * M + 1):][:2 * (2 * M + 1)].astype(LD)
    return s[0::2] + 1j * s[1::2]


# Chains of 11 to 86 modes (1, 2, 3, 4 and 6 tiles), both directions, steps all on the squaring side; Re low
# enough that the faster columns and modes fall below the rounding of the input.  Bar: the stepper's, some 16
# roundings of half an ulp in each of the steps: 8 steps eps of the majorant (FP32: plus what underflows).
@pytest.mark.parametrize("N,Re,steps,prec,adj", [
    (64, 5.0, 400, 0, False), (128, 20.0, 200, 0, False), (128, 20.0, 199, 0, True), (256, 20.0, 200, 0, False),
    (384, 40.0, 200, 0, True), (512, 60.0, 200, 0, False), (48, 5.0, 200, 1, True), (128, 20.0, 200, 1, False),
    (256, 20.0, 127, 1, True), (512, 60.0, 129, 1, False)])
def test_squared_chains_keep_damped_modes(tsk, N, Re, steps, prec, adj):
    print(f"damped chains N={N} Re={Re} steps={steps} prec={prec} adj={adj}", flush=True)
    op = _op(tsk, N, Re, prec, steps)
    tsk.set_base_kolmogorov(op, 4)
    x, y = _run(tsk, op, 21, adj)
    M = (N - 1) // 3
    eps, floor = (2.0 ** -52, 0.0) if prec == 0 else (2.0 ** -23, 1e-35)
    for kx in sorted({1, M // 4 + 1, M // 2 + 1, M}):
        xs, ys = _column(x, N, kx), _column(y, N, kx)
        for c in range(4):
            jy = np.arange(-M + (c + M) % 4, M + 1, 4)
            K2 = (LD(0.5) * kx) ** 2 + LD(1) * jy * jy
            g = LD(0.5) * (LD(0.5) * kx) * (1 - 16 / K2)
            S = _lawson(np.diag(g[1:], 1) - np.diag(g[:-1], -1), K2, Re)
            S = S.T if adj else S
            xc, got = xs[jy + M], ys[jy + M]
            want = xc
            for _ in range(steps):
                want = S @ want
            bar = 8 * steps * eps * _majorant(S, xc, steps) + floor
            assert np.all(np.abs(got - want) <= bar), (kx, c, float(np.max(np.abs(got - want) / bar)))
