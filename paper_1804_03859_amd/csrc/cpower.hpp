// Dense complex propagators by repeated squaring, batched over independent
// matrices.
//
// nsteps identical steps v <- S v + h of an n x n complex system (h = 0: a plain
// propagator) are taken by doubling: with S = I + D,
//     v <- v + D v + q     (2^k steps, applied for every set bit k of nsteps)
//     q <- 2 q + D q,  D <- 2 D + D D     (from 2^k to 2^(k+1) steps),
// q = h at k = 0.  Squaring D instead of S keeps the relative accuracy of the small
// step matrix.  After `squarings` doublings the last matrix is applied nsteps >>
// squarings times.
//
// Layout: real and imaginary planes, row-major, leading dimension ld (a multiple
// of 16, or of 32 for two tiles per wavefront), zero beyond n; two buffers that the
// doublings alternate between.  Vectors: four planes (v re, v im, q re, q im) per
// matrix, two buffers.
//
// k_cpow_gemm: one wavefront per MT x MT tiles of 16 x 16, four products
// v_mfma_{f64,f32}_16x16x4 per complex tile product; the fragments come straight
// from global memory (a lane's four A values are consecutive, the k index of MFMA r
// is 16 g + 4 (lane / 16) + r), the next 16 k loaded while the current ones
// multiply.  The matrices of a launch stay on one XCD each (its L2 then holds the
// operands of all its workgroups).  The vector updates of the same doubling
// read the same D, so they ride along as extra workgroups, one wavefront per row.
// Bound: the matrix cores (4 x 64 cycles per FP64 tile and 4 k), for few small
// matrices the launch and the load latency at its start.
#pragma once

#include "colpower.hpp"
#include "ops.hpp"

namespace tsk {

template <typename real> using vec4 = real __attribute__((ext_vector_type(4)));

enum CpowEpi {
    CPOW_SQUARE = 0,  // out = 2 A + A A
};

template <typename real> struct CpowArgs {
    const real* A;   // [count][2][ld * ld]
    const real* B;
    real* out;
    const real* vin;  // [count][4][ld]
    real* vout;
    int ld, count;
    int tile_blocks;  // workgroups of the tiles per matrix
    int bit, affine;  // vector updates of this doubling
};

// One row of the vector updates by one wavefront.
template <typename real>
__device__ inline void cpow_row(const real* __restrict__ D, int ld, int row, const real* __restrict__ vin, bool bit,
                                bool affine, real (&v)[4]) {
    const int lane = lane_id();
    const real* dr = D + size_t(row) * ld;
    const real* di = dr + size_t(ld) * ld;
    real s[4] = {real(0), real(0), real(0), real(0)};
    for (int k = lane; k < ld; k += kWave) {
        const real a = dr[k], b = di[k];
        if (bit) {
            const real x = vin[k], y = vin[ld + k];
            s[0] = fma(a, x, fma(-b, y, s[0]));
            s[1] = fma(a, y, fma(b, x, s[1]));
        }
        if (affine) {
            const real x = vin[2 * ld + k], y = vin[3 * ld + k];
            s[2] = fma(a, x, fma(-b, y, s[2]));
            s[3] = fma(a, y, fma(b, x, s[3]));
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < 2 ? bit : affine) {
            s[q] += xor_lane<32>(s[q], lane);
            s[q] += xor_lane<16>(s[q], lane);
            s[q] += xor_lane<8>(s[q], lane);
            s[q] += xor_lane<4>(s[q], lane);
            s[q] += xor_lane<2>(s[q], lane);
            s[q] += xor_lane<1>(s[q], lane);
        }
    }
    const real v0 = vin[row], v1 = vin[ld + row];
    const real q0 = affine ? vin[2 * ld + row] : real(0), q1 = affine ? vin[3 * ld + row] : real(0);
    v[0] = bit ? v0 + s[0] + q0 : v0;
    v[1] = bit ? v1 + s[1] + q1 : v1;
    v[2] = real(2) * q0 + s[2];
    v[3] = real(2) * q1 + s[3];
}

// Workgroup id -> (matrix, workgroup of the matrix): workgroups go to the 8 XCDs
// in turn, matrix m takes XCD m mod 8 (a single matrix: all of them).
__device__ inline void cpow_place(int id, int per, int count, int& m, int& w) {
    const int full = count / 8 * 8 * per;  // whole rounds of eight matrices
    if (id < full) {
        const int round = id / (8 * per), r = id % (8 * per);
        m = 8 * round + r % 8;
        w = r / 8;
    } else {
        const int left = count % 8, r = id - full;
        m = count / 8 * 8 + r % left;
        w = r / left;
    }
}

template <typename real, int MT, int EPI>
__global__ __launch_bounds__(4 * kWave) void k_cpow_gemm(CpowArgs<real> g) {
    using T = MfmaTile<real>;
    using V = typename T::V;
    const int ld = g.ld, wv = int(threadIdx.x) / kWave, lane = int(threadIdx.x) % kWave;
    const int vblocks = (g.bit || g.affine) ? ld / 4 : 0;
    int m, w;
    cpow_place(int(blockIdx.x), g.tile_blocks + vblocks, g.count, m, w);
    const size_t mat = size_t(ld) * ld;
    const real* A = g.A + 2 * mat * m;
    if (w >= g.tile_blocks) {
        const int row = 4 * (w - g.tile_blocks) + wv;
        real v[4];
        cpow_row<real>(A, ld, row, g.vin + size_t(4 * ld) * m, g.bit, g.affine, v);
        if (lane == 0) {
            real* o = g.vout + size_t(4 * ld) * m + row;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < 2 || g.affine) o[q * ld] = v[q];
        }
        return;
    }
    const real* B = g.B + 2 * mat * m;
    real* O = g.out + 2 * mat * m;
    constexpr int TS = 16 * MT;
    const int wt = (ld + 2 * TS - 1) / (2 * TS);
    const int r0 = (2 * (w / wt) + (wv >> 1)) * TS, c0 = (2 * (w % wt) + (wv & 1)) * TS;
    if (r0 >= ld || c0 >= ld) return;
    const int lr = lane & 15, lk = lane >> 4;
    const real* pa = A + size_t(r0 + lr) * ld + 4 * lk;
    const real* pb = B + size_t(4 * lk) * ld + c0 + lr;
    V accr[MT][MT], acci[MT][MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (EPI == CPOW_SQUARE) {
                    const size_t o = size_t(r0 + 16 * i + T::row(lane, r)) * ld + c0 + 16 * j + lr;
                    accr[i][j][r] = real(2) * A[o];
                    acci[i][j][r] = real(2) * A[o + mat];
                } else {
                    accr[i][j][r] = acci[i][j][r] = real(0);
                }
            }
    vec4<real> ar[MT], ai[MT];
    real br[MT][4], bi[MT][4];
    auto load = [&](int k, vec4<real> (&xr)[MT], vec4<real> (&xi)[MT], real (&yr)[MT][4], real (&yi)[MT][4]) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const real* p = pa + size_t(16 * i) * ld + k;
            xr[i] = *reinterpret_cast<const vec4<real>*>(p);
            xi[i] = *reinterpret_cast<const vec4<real>*>(p + mat);
        }
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const real* p = pb + size_t(k + r) * ld + 16 * j;
                yr[j][r] = p[0];
                yi[j][r] = p[mat];
            }
    };
    load(0, ar, ai, br, bi);
    for (int k = 0; k < ld; k += 16) {
        vec4<real> nar[MT], nai[MT];
        real nbr[MT][4], nbi[MT][4];
        load(k + 16 < ld ? k + 16 : k, nar, nai, nbr, nbi);  // in flight during the products below
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    accr[i][j] = T::fma(ar[i][r], br[j][r], accr[i][j]);
                    acci[i][j] = T::fma(ar[i][r], bi[j][r], acci[i][j]);
                    accr[i][j] = T::fma(-ai[i][r], bi[j][r], accr[i][j]);
                    acci[i][j] = T::fma(ai[i][r], br[j][r], acci[i][j]);
                }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            ar[i] = nar[i];
            ai[i] = nai[i];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                br[i][r] = nbr[i][r];
                bi[i][r] = nbi[i][r];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const size_t o = size_t(r0 + 16 * i + T::row(lane, r)) * ld + c0 + 16 * j + lr;
                O[o] = accr[i][j][r];
                O[o + mat] = acci[i][j][r];
            }
}

// Where the result of a matrix goes: interleaved complex values at base + m stride,
// or at table[m]; rows 0 .. n - 1.
template <typename real> struct CpowOut {
    real* base;
    int64_t stride;
    real* const* table;
    int n;
};

// v <- v + D v + q; last: to the caller's output instead of vout.
template <typename real>
__global__ __launch_bounds__(4 * kWave) void k_cpow_apply(CpowArgs<real> g, CpowOut<real> out, int last) {
    const int ld = g.ld, wv = int(threadIdx.x) / kWave, lane = int(threadIdx.x) % kWave;
    int m, w;
    cpow_place(int(blockIdx.x), ld / 4, g.count, m, w);
    const int row = 4 * w + wv;
    const real* vin = g.vin + size_t(4 * ld) * m;
    real v[4];
    cpow_row<real>(g.A + 2 * size_t(ld) * ld * m, ld, row, vin, true, false, v);
    if (g.affine) {
        v[0] += vin[2 * ld + row];
        v[1] += vin[3 * ld + row];
    }
    if (lane != 0) return;
    if (last) {
        if (row < out.n) {
            real* y = out.table ? out.table[m] : out.base + out.stride * m;
            y[2 * row] = v[0];
            y[2 * row + 1] = v[1];
        }
    } else {
        real* o = g.vout + size_t(4 * ld) * m + row;
        o[0] = v[0];
        o[ld] = v[1];
        if (g.affine) {
            o[2 * ld] = vin[2 * ld + row];
            o[3 * ld] = vin[3 * ld + row];
        }
    }
}

// Workspace of `count` matrices: two buffers of matrices and of vectors.
struct CpowWork {
    DevBuf mat, vec;
    int count = 0, ld = 0, mt = 1;
    size_t real_bytes = 8;
    // Bytes per matrix (both buffers).
    static size_t bytes(int ld, size_t rb) { return 4 * size_t(ld) * ld * rb; }
    template <typename real> real* D(int b) const { return mat.as<real>() + size_t(b) * 2 * ld * ld * count; }
    template <typename real> real* v(int b) const { return vec.as<real>() + size_t(b) * 4 * ld * count; }
    bool fits(int n_, int count_, size_t rb) const {
        return mat.ptr && ld >= n_ && count == count_ && real_bytes == rb;
    }
    tsk_status ensure(int n_, int count_, size_t rb) {
        // two tiles per wavefront once one tile each would queue several wavefronts per SIMD
        const int t = (n_ + 15) / 16;
        mt = double(t) * t * count_ >= 3072.0 ? 2 : 1;
        ld = (n_ + 16 * mt - 1) / (16 * mt) * (16 * mt);
        count = count_;
        real_bytes = rb;
        TSK_TRY(mat.ensure(bytes(ld, rb) * count));
        return vec.ensure(8 * size_t(ld) * rb * count);
    }
};

// Doublings before the last matrix is applied nsteps >> k times: one more has to
// save more applications than it costs.  ratio: cost of a doubling over that of an
// application.
inline int cpow_doublings(int64_t nsteps, double ratio) {
    int k = 0;
    while (double((nsteps >> k) - (nsteps >> (k + 1))) > ratio) ++k;
    return k;
}

// The nsteps steps of the matrices in W.D(0) and vectors in W.v(0).
template <typename real>
tsk_status cpow_run(const CpowWork& W, int64_t nsteps, bool affine, int doublings, const CpowOut<real>& out,
                    hipStream_t s) {
    const int ld = W.ld, ts = 32 * W.mt, wt = (ld + ts - 1) / ts;
    int b = 0, vb = 0;
    for (int k = 0; k < doublings; ++k) {
        CpowArgs<real> g{};
        g.A = g.B = W.D<real>(b);
        g.out = W.D<real>(b ^ 1);
        g.vin = W.v<real>(vb);
        g.vout = W.v<real>(vb ^ 1);
        g.ld = ld;
        g.count = W.count;
        g.tile_blocks = wt * wt;
        g.bit = int((nsteps >> k) & 1);
        g.affine = affine ? 1 : 0;
        const int vblocks = (g.bit || g.affine) ? ld / 4 : 0;
        const dim3 grid(unsigned((g.tile_blocks + vblocks) * W.count));
        if (W.mt == 2)
            hipLaunchKernelGGL((k_cpow_gemm<real, 2, CPOW_SQUARE>), grid, dim3(4 * kWave), 0, s, g);
        else
            hipLaunchKernelGGL((k_cpow_gemm<real, 1, CPOW_SQUARE>), grid, dim3(4 * kWave), 0, s, g);
        b ^= 1;
        if (vblocks) vb ^= 1;
    }
    for (int64_t r = nsteps >> doublings; r > 0; --r) {
        CpowArgs<real> g{};
        g.A = W.D<real>(b);
        g.vin = W.v<real>(vb);
        g.vout = W.v<real>(vb ^ 1);
        g.ld = ld;
        g.count = W.count;
        g.affine = affine ? 1 : 0;
        hipLaunchKernelGGL(k_cpow_apply<real>, dim3(unsigned(ld / 4 * W.count)), dim3(4 * kWave), 0, s, g, out,
                           r == 1 ? 1 : 0);
        vb ^= 1;
    }
    TSK_HIP(hipGetLastError());
    return TSK_OK;
}

}  // namespace tsk
