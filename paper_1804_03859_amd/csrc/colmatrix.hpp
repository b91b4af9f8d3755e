// Time integration about a parallel base flow by repeated squaring of each kx
// column's one-step matrix (cpower.hpp), for profiles that are not one harmonic.
//
// In the kx column the advection term of the pseudo-spectral product is a matrix on
// the kept modes ky = -M..M,
//     A_ij = i (-U^_{i-j} kx + O^_{i-j} kx / K_j^2),
// U^_m, O^_m the N-point DFT coefficients (1/N) sum_l f_l e^{-2 pi i m l / N} of U and
// dOmega/dy, the index taken mod N (the products that wrap on the grid are the
// operator's too).  A Lawson RK4 step is a polynomial in A and the diagonal
// integrating factors: three products form S - diag(b) (the STAGE epilogues, b as in cpower.hpp), then the
// powers follow as in cpower.hpp, all columns together.  A profile of harmonics up to h
// makes A banded (h off the diagonal, 4 h the step), and the products stay inside the
// band.  The column stepper takes nsteps x 4 dependent stages of three transforms
// on one wavefront per column.
#pragma once

#include "colstep.hpp"
#include "cpower.hpp"

namespace tsk {

// A into `A`, its rows scaled by eh into `X`, the diagonal factors into `diag`, b of the
// one-step matrix (cpower.hpp) behind `C`, the input columns into `vec` (q = 0); the
// workgroups of matrix index M advance the kx = 0 column.  prof: [N][4] (U^ re, im, O^ re, im).  Grid x: row, grid y: column
// kx - 1 (0 .. M).
template <typename real>
__global__ __launch_bounds__(4 * kWave) void k_colmatrix_form(ColInst<real> I, const double* __restrict__ prof, int N,
                                                              int ld, real* __restrict__ A, real* __restrict__ X,
                                                              double* __restrict__ diag, real* __restrict__ vec,
                                                              real* __restrict__ C) {
    const int M = I.M, NM = 2 * M + 1, row = int(blockIdx.x), m = int(blockIdx.y), tid = int(threadIdx.x);
    if (m == M) {
        for (int q = row * int(blockDim.x) + tid; q < M; q += int(gridDim.x * blockDim.x)) {
            const double jy = q + 1, E = exp(-jy * jy * I.dt / I.Re * I.nsteps);
            I.y[2 * q] = real(E * double(I.xbase[2 * q]));
            I.y[2 * q + 1] = real(E * double(I.xbase[2 * q + 1]));
        }
        return;
    }
    const double kxv = I.alpha * (m + 1);
    const size_t mat = size_t(ld) * ld;
    real* Am = A + cpow_stride(ld) * m + size_t(row) * ld;
    real* Xm = X + cpow_stride(ld) * m + size_t(row) * ld;
    const double ji = row - M, Ki = kxv * kxv + ji * ji;
    const bool kept = row < NM;
    const double ehq = -Ki * (0.5 * I.dt) / I.Re, ehm = kept ? expm1(ehq) : -1.0;
    const double eh = ehm > -0.5 ? 1.0 + ehm : kept ? exp(ehq) : 0.0;
    for (int c = tid; c < ld; c += int(blockDim.x)) {
        double ar = 0.0, ai = 0.0;
        if (kept && c < NM) {
            const double jc = c - M, g1 = kxv, g2 = kxv / (kxv * kxv + jc * jc);
            const int d = (row - c + 2 * N) % N;
            const double* p = prof + 4 * d;
            ar = -(-p[1] * g1 + p[3] * g2);  // i (re + i im) = -im + i re
            ai = -p[0] * g1 + p[2] * g2;
        }
        Am[c] = real(ar);
        Am[mat + c] = real(ai);
        Xm[c] = real(eh * ar);
        Xm[mat + c] = real(eh * ai);
    }
    if (tid == 0) {
        double* dg = diag + size_t(3 * ld) * m;
        const double e1m = ehm * (2.0 + ehm), e1 = e1m > -0.5 ? 1.0 + e1m : eh * eh;
        dg[row] = kept ? e1 : 0.0;
        dg[ld + row] = kept ? eh : 0.0;
        dg[2 * ld + row] = !kept ? 0.0 : e1m > -0.5 ? e1m : e1;
        C[cpow_stride(ld) * m + 2 * mat + row] = kept && e1m > -0.5 ? real(1) : real(0);
        real* v = vec + size_t(4 * ld) * m;
        const real* xs = I.xbase + 2ll * M + int64_t(m) * 2 * NM;
        v[row] = kept ? xs[2 * row] : real(0);
        v[ld + row] = kept ? xs[2 * row + 1] : real(0);
        v[2 * ld + row] = v[3 * ld + row] = real(0);
    }
}

// Blocks of 16 mt off the diagonal of a matrix with entries up to `width` off it.
inline int band_blocks(int width, int mt) { return (width + 16 * mt - 1) / (16 * mt); }

// One matvec (adj: of the transposed propagator) of the instance I, harmonics up to h.
template <typename real>
tsk_status colmatrix_run(const CpowWork& W, const ColInst<real>& I, const double* prof, int N, int h, bool adj,
                         int doublings, hipStream_t s) {
    const int ld = W.ld, M = I.M, NM = 2 * M + 1;
    double* diag = W.diag();
    hipLaunchKernelGGL(k_colmatrix_form<real>, dim3(ld, M + 1), dim3(4 * kWave), 0, s, I, prof, N, ld, W.D<real>(0),
                       W.D<real>(1), diag, W.v<real>(0), W.D<real>(2));
    const int ts = 32 * W.mt, wt = (ld + ts - 1) / ts;
    CpowArgs<real> g{};
    g.A = W.D<real>(0);
    g.ld = ld;
    g.count = M;
    g.tile_blocks = wt * wt;
    g.sum = W.D<real>(3);
    g.diag = diag;
    g.h = I.dt;
    g.adj = adj ? 1 : 0;
    const dim3 grid(unsigned(g.tile_blocks * M));
    // (the sum is read over the wider bands of the later stages: all of them one width)
    g.band_a = band_blocks(h, W.mt);
    g.band_c = band_blocks(4 * h, W.mt);
    g.B = W.D<real>(1);
    g.out = W.D<real>(2);
    g.band_b = g.band_a;
    cpow_gemm<real, CPOW_STAGE2>(W, grid, g, s);
    g.B = W.D<real>(2);
    g.out = W.D<real>(1);
    g.band_b = g.band_c;
    cpow_gemm<real, CPOW_STAGE3>(W, grid, g, s);
    g.B = W.D<real>(1);
    g.out = W.D<real>(2);
    cpow_gemm<real, CPOW_STAGE4>(W, grid, g, s);
    const CpowOut<real> out{I.y + 2ll * M, 2ll * NM, nullptr, NM};
    return cpow_run<real>(W, I.nsteps, false, g.band_c, doublings, out, s);
}

}  // namespace tsk
