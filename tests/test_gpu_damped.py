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


def _column_generator(U, d, kx):
    """Advection matrix of a kx column on the kept modes, from the samples the operator holds."""
    N = len(U)
    M = (N - 1) // 3
    ky = np.arange(-M, M + 1)
    F = np.exp(-1j * (2 * np.arctan2(LD(0), LD(-1)) / N) *
               (np.arange(N)[:, None] * np.arange(N)[None, :] % N).astype(LD))
    u, o = F @ U.astype(LD) / N, F @ d.astype(LD) / N
    k = LD(0.5) * kx
    K2 = k * k + LD(1) * ky * ky
    D = (ky[:, None] - ky[None, :]) % N
    return 1j * (-u[D] * k + o[D] * k / K2[None, :]), K2


# Whole columns (16, 32, 48, 64 and, two tiles per wavefront, 128 modes padded), narrow and full bands.  The column
# stepper transforms a column at a time, so its bar is one of norms: 8 steps eps max_q |S^(n-q)| |S^q| |x|.
@pytest.mark.parametrize("N,Re,steps,base,adj,prec", [
    (16, 0.5, 200, "wide", False, 0), (32, 1.0, 200, "narrow", True, 0), (64, 5.0, 400, "narrow", False, 0),
    (96, 10.0, 200, "wide", True, 0), (192, 10.0, 200, "narrow", False, 0), (32, 1.0, 200, "wide", False, 1),
    (192, 20.0, 100, "narrow", True, 1)])
def test_squared_columns_keep_damped_columns(tsk, N, Re, steps, base, adj, prec):
    print(f"damped columns N={N} Re={Re} steps={steps} base={base} adj={adj} prec={prec}", flush=True)
    y = 2 * np.pi * np.arange(N) / N
    hs = ((1, 0.7), (2, 0.3)) if base == "narrow" else ((1, 0.6), (N // 5, 0.02), (N // 3 + 1, 0.002))
    U = sum(a * np.sin(h * y + 0.3 * h) for h, a in hs)
    d = sum(a * h * h * np.sin(h * y + 0.3 * h) for h, a in hs)
    op = _op(tsk, N, Re, prec, steps)
    tsk.set_base_parallel(op, U, d)
    xin, yout = _run(tsk, op, 22, adj)
    M = (N - 1) // 3
    eps, floor = (2.0 ** -52, 0.0) if prec == 0 else (2.0 ** -23, 1e-35)
    norm = lambda v: float(np.linalg.norm(v.astype(complex), 2))  # noqa: E731
    for kx in sorted({1, M // 2 + 1, M}):
        A, K2 = _column_generator(U, d, kx)
        S = _lawson(A, K2, Re)
        S = S.conj().T if adj else S
        xc, got = _column(xin, N, kx), _column(yout, N, kx)
        want, P8 = xc, _power(S, steps // 8)
        for _ in range(steps):
            want = S @ want
        powers = [norm(_power(P8, q)) for q in range(9)]
        grow = max(powers[q] * powers[8 - q] for q in range(9))
        bar = 8 * steps * eps * grow * norm(xc) + floor
        assert norm(got - want) <= bar, (kx, norm(got - want) / bar)


# A Ginzburg-Landau propagator below the threshold everywhere (mu0 = -1.5): the state decays by e^(-1.5 T) and more.
# Bar as above, in the largest norm; the step matrix in extended precision.
@pytest.mark.parametrize("n,hw,steps,adj", [(16, 20.0, 3000, False), (60, 20.0, 2000, True), (130, 30.0, 2500, False)])
def test_squared_ginzburg_landau_keeps_decayed_states(tsk, n, hw, steps, adj):
    print(f"damped cgle n={n} steps={steps} adj={adj}", flush=True)
    from oracle.cgle import CGLE
    par = dict(U=2.0, c_u=0.2, c_d=-1.0, mu0=-1.5, mu2=-0.01)
    ref = CGLE(n=n, half_width=hw, dt=0.01, T=0.01 * steps, **par)
    op = tsk.create_cgle1d(n, hw)
    tsk.set_params_cgle(op, par["U"], par["c_u"], par["c_d"], par["mu0"], par["mu2"], 0.01, 0.01 * steps)
    u = W.cgle_start(n, 5)
    x = torch.from_numpy(u).cuda()
    y = torch.zeros_like(x)
    (tsk.apply_adjoint if adj else tsk.apply)(op, x, y)
    L = ref.matrix().astype(CLD)
    L = L.conj().T if adj else L
    h = LD(0.01) / 2
    lhs, rhs = np.eye(n) - h * L, np.eye(n) + h * L
    B = rhs.copy()  # (I - h L)^-1 (I + h L) by elimination (diagonally dominant, tridiagonal)
    T = lhs.copy()
    for i in range(1, n):
        f = T[i, i - 1] / T[i - 1, i - 1]
        T[i] -= f * T[i - 1]
        B[i] -= f * B[i - 1]
    for i in range(n - 1, -1, -1):
        if i + 1 < n:
            B[i] -= T[i, i + 1] * B[i + 1]
        B[i] /= T[i, i]
    want = u.astype(CLD)
    for _ in range(steps):
        want = B @ want
    bar = 8 * steps * 2.0 ** -52 * np.max(_majorant(B, u.astype(CLD), steps))
    err = np.max(np.abs(y.cpu().numpy().astype(CLD) - want))
    assert err <= bar, float(err / bar)
    assert np.max(np.abs(want)) < 1e-12 * np.max(np.abs(u))
