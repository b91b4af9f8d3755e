// Dense complex propagators by repeated squaring, batched over independent
// matrices.
//
// nsteps identical steps v <- S v + h of an n x n complex system (h = 0: a plain
// propagator) are taken by doubling: with S = diag(b) + C,
//     v <- b v + C v + q     (2^k steps, applied for every set bit k of nsteps)
//     q <- (1 + b) q + C q,  C_ij <- (b_i + b_j) C_ij + (C C)_ij     (to 2^(k+1) steps),
// q = h at k = 0.  b = 1 where the diagonal entry of S is near 1: C = S - I there, which
// keeps the relative accuracy of the small step matrix.  Once that entry is below 1/2
// in modulus, b turns to 0 and C holds S itself: s - 1 would lose a damped mode (as in
// colpower.hpp).  After `squarings` doublings the last matrix is applied nsteps >>
// squarings times.
//
// Layout: real and imaginary planes, row-major, leading dimension ld (a multiple
// of 16, or of 32 for two tiles per wavefront), zero beyond n, and b behind them; two
// buffers that the doublings alternate between.  Vectors: four planes (v re, v im, q re, q im) per
// matrix, two buffers.
//
// Bands: a matrix whose entries vanish beyond a distance from the diagonal is stored
// with only its blocks |bi - bj| <= band valid (blocks of 16 MT, what one wavefront
// computes; ld / (16 MT) or more: all), and a doubling doubles the band; blocks
// outside are neither written nor read.
//
// k_cpow_gemm: one wavefront per MT x MT tiles of 16 x 16, four products
// v_mfma_{f64,f32}_16x16x4 per complex tile product; the fragments come straight
// from global memory (a lane's four A values are consecutive, the k index of MFMA r
// is 16 g + 4 (lane / 16) + r), the next 16 or 48 k loaded while the current ones
// multiply.  The matrices of a launch stay on one XCD each (its L2 then holds the
// operands of all its workgroups).  The vector updates of the same doubling
// read the same D, so they ride along as extra workgroups, one wavefront per row.
// Bound: the matrix cores (4 x 64 cycles per FP64 tile and 4 k), for few small
// matrices the launch and the load latency at its start.  One doubling, FP64, as traced: one
// matrix of 256 16.5 us, of 400 23.7, of 1000 138; 42 of 85 (dense) 14.5, 63 of 127 26
// with the vector rows, 85 of 171 90 (38 TFLOP/s).  The rows launched between the tiles
// instead of after them: 42 against 31 for the 63.
#pragma once

#include <algorithm>

#include "colpower.hpp"
#include "ops.hpp"

namespace tsk {

template <typename real> using vec4 = real __attribute__((ext_vector_type(4)));

// Products G = A B of k_cpow_gemm.  CPOW_SQUARE: out = (b_i + b_j) A + G (B = A).  The
// other three form C of a Lawson RK4 step from the advection matrix A (column j's unit
// vector through the four stages, diagonal factors e1 = E(h), eh = E(h/2)):
//     STAGE2: t = A_ij eh_j + h/2 G,  sum = e1_i A_ij + 2 eh_i t,  out = t
//     STAGE3: t = A_ij eh_j + h/2 G,  sum += 2 eh_i t,             out = eh_i t
//     STAGE4: t = A_ij e1_j + h G,    out = (e1 - b) I + h/6 (sum + t)
enum CpowEpi { CPOW_SQUARE = 0, CPOW_STAGE2, CPOW_STAGE3, CPOW_STAGE4 };

// Reals of a matrix: two planes, and b behind them.
__host__ __device__ inline size_t cpow_stride(int ld) { return 2 * size_t(ld) * ld + ld; }

template <typename real> struct CpowArgs {
    const real* A;   // [count][cpow_stride]
    const real* B;
    real* out;
    const real* vin;  // [count][4][ld]
    real* vout;
    int ld, count;
    int band_a, band_b, band_c;  // blocks off the diagonal
    int tile_blocks;  // workgroups of the tiles per matrix
    int ts;           // k_cpow_apply: 16 MT
    int bit, affine;  // vector updates of this doubling
    // stages only
    real* sum;
    const double* diag;  // [count][3][ld]: e1, eh, e1 - b
    double h;
    int adj;  // STAGE4: the conjugate transpose of C
};

// One row of the vector updates by one wavefront.
template <typename real>
__device__ inline void cpow_row(const real* __restrict__ D, int ld, int ts, int band, int row,
                                const real* __restrict__ vin, bool bit, bool affine, real (&v)[4]) {
    const int lane = lane_id();
    const real* dr = D + size_t(row) * ld;
    const real* di = dr + size_t(ld) * ld;
    real s[4] = {real(0), real(0), real(0), real(0)};
    const real v0 = vin[row], v1 = vin[ld + row], b = D[2 * size_t(ld) * ld + row];  // under the sum's latency
    const int lo = max(0, ts * (row / ts - band)), hi = min(ld, ts * (row / ts + band + 1));
    for (int k = lo + lane; k < hi; k += kWave) {
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
    const real q0 = affine ? vin[2 * ld + row] : real(0), q1 = affine ? vin[3 * ld + row] : real(0);
    v[0] = bit ? fma(b, v0, s[0]) + q0 : v0;
    v[1] = bit ? fma(b, v1, s[1]) + q1 : v1;
    v[2] = fma(real(1) + b, q0, s[2]);
    v[3] = fma(real(1) + b, q1, s[3]);
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

// Two wavefronts per SIMD as the occupancy floor caps the kernel at 256 registers, where
// the compiler keeps the accumulators in plain vector registers.  Without it they sit
// in the accumulation half and move out and back around the products (MT = 2: 5 to
// 15 % slower, MT = 1 the same).
template <typename real, int MT, int EPI>
__global__ __launch_bounds__(4 * kWave, 2) void k_cpow_gemm(CpowArgs<real> g) {
    using T = MfmaTile<real>;
    using V = typename T::V;
    const int ld = g.ld, wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
    const int lane = int(threadIdx.x) % kWave;
    // the tiles of all matrices first: the rows fill in beside them
    int m, w;
    const int ntile = g.tile_blocks * g.count;
    const bool rows = int(blockIdx.x) >= ntile;
    if (rows)
        cpow_place(int(blockIdx.x) - ntile, ld / 4, g.count, m, w);
    else
        cpow_place(int(blockIdx.x), g.tile_blocks, g.count, m, w);
    const size_t mat = size_t(ld) * ld;
    const real* A = g.A + cpow_stride(ld) * m;
    if (rows) {
        const int row = 4 * w + wv;
        real v[4];
        cpow_row<real>(A, ld, 16 * MT, g.band_a, row, g.vin + size_t(4 * ld) * m, g.bit, g.affine, v);
        if (lane == 0) {
            real* o = g.vout + size_t(4 * ld) * m + row;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < 2 || g.affine) o[q * ld] = v[q];
        }
        return;
    }
    const real* B = g.B + cpow_stride(ld) * m;
    real* O = g.out + cpow_stride(ld) * m;
    constexpr int TS = 16 * MT;
    const int wt = (ld + 2 * TS - 1) / (2 * TS);
    const int r0 = (2 * (w / wt) + (wv >> 1)) * TS, c0 = (2 * (w % wt) + (wv & 1)) * TS;
    if (r0 >= ld || c0 >= ld) return;
    // the wavefront's block, and the k range inside both bands
    const int rt = r0 / TS, ct = c0 / TS, off = rt > ct ? rt - ct : ct - rt;
    if (off > g.band_c) return;
    const int kfirst = max(0, max(rt - g.band_a, ct - g.band_b)) * TS;
    const int kend = min(ld, min(rt + 1 + g.band_a, ct + 1 + g.band_b) * TS);
    const int lr = lane & 15, lk = lane >> 4;
    // uniform row pointers plus 32-bit lane offsets: the loads take the scalar-base
    // form and the address arithmetic stays off the vector unit
    const unsigned oa = unsigned(lr) * unsigned(ld) + 4u * unsigned(lk);
    const unsigned ob = 4u * unsigned(lk) * unsigned(ld) + unsigned(lr);
    const real* pa = A + size_t(r0) * ld;
    const real* pb = B + c0;
    V accr[MT][MT], acci[MT][MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) accr[i][j][r] = acci[i][j][r] = real(0);
    // ST stages of 16 k in registers: while one multiplies, the next ST - 1 load
    constexpr int ST = MT == 1 ? 4 : 2;
    vec4<real> ar[ST][MT], ai[ST][MT];
    real br[ST][MT][4], bi[ST][MT][4];
    auto load = [&](int st, int k) {
        k = k < kend ? k : kend - 16;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const real* p = pa + size_t(16 * i) * ld + k;
            ar[st][i] = *reinterpret_cast<const vec4<real>*>(p + oa);
            ai[st][i] = *reinterpret_cast<const vec4<real>*>(p + mat + oa);
        }
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const real* p = pb + size_t(k + r) * ld + 16 * j;
                br[st][j][r] = p[ob];
                bi[st][j][r] = (p + mat)[ob];
            }
    };
    auto products = [&](int st) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    accr[i][j] = T::fma(ar[st][i][r], br[st][j][r], accr[i][j]);
                    acci[i][j] = T::fma(ar[st][i][r], bi[st][j][r], acci[i][j]);
                    accr[i][j] = T::fma(-ai[st][i][r], bi[st][j][r], accr[i][j]);
                    acci[i][j] = T::fma(ai[st][i][r], br[st][j][r], acci[i][j]);
                }
    };
#pragma unroll
    for (int st = 0; st < ST - 1; ++st) load(st, kfirst + 16 * st);
    int k0 = kfirst;
    for (; k0 + 16 * ST <= kend; k0 += 16 * ST) {
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            load((st + ST - 1) % ST, k0 + 16 * (st + ST - 1));
            // keeps the loads here, ahead of the products (the compiler would sink
            // them to their uses)
            __builtin_amdgcn_sched_barrier(0);
            products(st);
        }
    }
    // CPOW_SQUARE's (b_i + b_j) A, loaded under the last products and added to their sum:
    // products added to it one after the other would each be rounded at its size (256
    // nodes, 9000 steps: error against long double 3e-13, so 1e-13).  Every wavefront
    // loads the values that only some use (blocks outside the band, the diagonal) and
    // selects: a branch would wait for each load in turn.
    constexpr int SQ = EPI == CPOW_SQUARE ? MT : 1;
    real cx[SQ][SQ][4], cy[SQ][SQ][4], rb[SQ][4], cb[SQ], dx[SQ], dy[SQ];
    if constexpr (EPI == CPOW_SQUARE) {
        const real* bm = A + 2 * mat;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int ri = r0 + 16 * i + lr;
            cb[i] = bm[c0 + 16 * i + lr];
            dx[i] = A[size_t(ri) * ld + ri];
            dy[i] = A[size_t(ri) * ld + ri + mat];
#pragma unroll
            for (int r = 0; r < 4; ++r) rb[i][r] = bm[r0 + 16 * i + T::row(lane, r)];
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const size_t o = size_t(r0 + 16 * i + T::row(lane, r)) * ld + c0 + 16 * j + lr;
                    cx[i][j][r] = A[o];
                    cy[i][j][r] = A[o + mat];
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int st = 0; st < ST - 1; ++st)  // the last ld / 16 mod ST stages, already loaded
        if (k0 + 16 * st < kend) products(st);
    if constexpr (EPI == CPOW_SQUARE) {
        const bool inside = off <= g.band_a;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            // the diagonal: b of the square, judged by the square of the entry (cb is b there)
            const real x = real(1) + dx[i], y = dy[i];
            const bool turn = off == 0 && cb[i] != real(0) && x * x + y * y < real(0.5);
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const real b = rb[i][r] + cb[j];
                    const real one = i == j && turn && T::row(lane, r) == lr ? real(1) : real(0);
                    accr[i][j][r] += inside ? fma(b, cx[i][j][r], one) : real(0);
                    acci[i][j][r] += inside ? b * cy[i][j][r] : real(0);
                }
            if (off == 0 && lane < 16) O[2 * mat + r0 + 16 * i + lr] = turn ? real(0) : cb[i];
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const size_t o = size_t(r0 + 16 * i + T::row(lane, r)) * ld + c0 + 16 * j + lr;
                if constexpr (EPI == CPOW_SQUARE) {
                    O[o] = accr[i][j][r];
                    O[o + mat] = acci[i][j][r];
                } else {
                    const int ri = r0 + 16 * i + T::row(lane, r), cj = c0 + 16 * j + lr;
                    const double* dg = g.diag + size_t(3 * ld) * m;
                    const double ej = EPI == CPOW_STAGE4 ? dg[cj] : dg[ld + cj];
                    const double hc = EPI == CPOW_STAGE4 ? g.h : 0.5 * g.h, e1i = dg[ri], ehi = dg[ld + ri];
                    real* sm = g.sum + cpow_stride(ld) * m;
                    const double ax = A[o], ay = A[o + mat];
                    const double bx = ax * ej + hc * double(accr[i][j][r]), by = ay * ej + hc * double(acci[i][j][r]);
                    if constexpr (EPI == CPOW_STAGE2) {
                        sm[o] = real(e1i * ax + 2.0 * ehi * bx);
                        sm[o + mat] = real(e1i * ay + 2.0 * ehi * by);
                        O[o] = real(bx);
                        O[o + mat] = real(by);
                    } else if constexpr (EPI == CPOW_STAGE3) {
                        sm[o] = real(double(sm[o]) + 2.0 * ehi * bx);
                        sm[o + mat] = real(double(sm[o + mat]) + 2.0 * ehi * by);
                        O[o] = real(ehi * bx);
                        O[o + mat] = real(ehi * by);
                    } else {
                        const double h6 = g.h / 6.0;
                        const double dx = h6 * (double(sm[o]) + bx) + (ri == cj ? dg[2 * ld + ri] : 0.0);
                        const double dy = h6 * (double(sm[o + mat]) + by);
                        const size_t p = g.adj ? size_t(cj) * ld + ri : o;
                        O[p] = real(dx);
                        O[p + mat] = real(g.adj ? -dy : dy);
                    }
                }
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

// v <- b v + C v + q; last: to the caller's output instead of vout.
template <typename real>
__global__ __launch_bounds__(4 * kWave) void k_cpow_apply(CpowArgs<real> g, CpowOut<real> out, int last) {
    const int ld = g.ld, wv = int(threadIdx.x) / kWave, lane = int(threadIdx.x) % kWave;
    int m, w;
    cpow_place(int(blockIdx.x), ld / 4, g.count, m, w);
    const int row = 4 * w + wv;
    const real* vin = g.vin + size_t(4 * ld) * m;
    real v[4];
    cpow_row<real>(g.A + cpow_stride(ld) * m, ld, g.ts, g.band_a, row, vin, true, false, v);
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

// The arrays of one call on `count` matrices, laid out in scratch memory (held while this
// lives: until the call has enqueued its launches): nbuf buffers of
// matrices (the doublings alternate between `first` and `first` ^ 1), two of vectors and
// the diagonal factors of the stages.
struct CpowWork {
    std::unique_lock<std::mutex> lock;
    char* base = nullptr;
    int count = 0, ld = 0, mt = 1, nbuf = 2, first = 0;
    size_t rb = 8;
    // Bytes per matrix and buffer.
    static size_t bytes(int ld, size_t rb) { return cpow_stride(ld) * rb; }
    template <typename real> real* D(int b) const {
        return reinterpret_cast<real*>(base) + size_t(b) * cpow_stride(ld) * count;
    }
    template <typename real> real* v(int b) const { return D<real>(nbuf) + size_t(b) * 4 * ld * count; }
    // (behind nbuf strides and 8 ld reals per matrix: a multiple of 16 reals)
    double* diag() const { return reinterpret_cast<double*>(base + nbuf * bytes(ld, rb) * count + 8 * ld * rb * count); }
    size_t total() const { return (nbuf * bytes(ld, rb) + 8 * ld * rb + 3 * ld * sizeof(double)) * count; }
    // Leading dimension and tiles per wavefront of `count` n x n matrices: two tiles per
    // wavefront once one each would queue several wavefronts per SIMD (63 matrices of
    // 127: a doubling 26 us with two, 36 with one; 42 of 85: 18 and 14).
    static int tiles_of(int n_, int count_) {
        const int t = (n_ + 15) / 16;
        return double(t) * t * count_ >= 3072.0 ? 2 : 1;
    }
    static int ld_of(int n_, int count_) {
        const int w = 16 * tiles_of(n_, count_);
        return (n_ + w - 1) / w * w;
    }
    // For launches on `stream`, or false: step instead (Scratch::get).
    bool place(Scratch& s, hipStream_t stream, int n_, int count_, size_t rb_, int nbuf_, int first_) {
        if (lock.owns_lock()) lock.unlock();
        lock = std::unique_lock<std::mutex>(s.mu);
        count = count_;
        mt = tiles_of(n_, count_);
        ld = ld_of(n_, count_);
        rb = rb_;
        nbuf = nbuf_;
        first = first_;
        base = static_cast<char*>(s.get(total(), stream));
        if (!base) lock.unlock();
        return base != nullptr;
    }
};

// Estimated times in us of the work on `count` matrices of leading dimension ld, MT tiles
// per wavefront, `band` blocks wide.
struct CpowCost {
    int ld, count, mt;
    bool fp32;
    double width(double band) const { return std::min(double(ld), 16.0 * mt * (2.0 * band + 1.0)); }
    // A product of matrices a and b wide: a launch and the loads' latency, or the
    // matrix cores.
    double product(double a, double b) const {
        const double k = std::min(width(a), width(b)), flops = 8.0 * ld * width(a + b) * k * count;
        return 2.8 + 0.045 * std::min(k, 256.0) + flops / (fp32 ? 1.0e8 : 6.0e7);
    }
    // An application: a launch, or the matrices' bytes.
    double application(double b) const {
        return 2.8 + (fp32 ? 8.0 : 16.0) * width(b) * ld * count / 7.0e6;
    }
    // The doublings k before the last matrix is applied nsteps >> k times that take the
    // least time, and that time.
    int doublings(int64_t nsteps, double band, double* cost) const {
        double spent = 0.0, best = 0.0;
        int bk = 0;
        for (int k = 0; k == 0 || (nsteps >> k) > 0; ++k, band *= 2.0) {
            const double total = spent + double(nsteps >> k) * application(band);
            if (k == 0 || total < best) {
                best = total;
                bk = k;
            }
            spent += product(band, band);
        }
        *cost = best;
        return bk;
    }
};

template <typename real, int EPI>
void cpow_gemm(const CpowWork& W, dim3 grid, const CpowArgs<real>& g, hipStream_t s) {
    if (W.mt == 2)
        hipLaunchKernelGGL((k_cpow_gemm<real, 2, EPI>), grid, dim3(4 * kWave), 0, s, g);
    else
        hipLaunchKernelGGL((k_cpow_gemm<real, 1, EPI>), grid, dim3(4 * kWave), 0, s, g);
}

// The nsteps steps of the matrices in W.D(W.first), `band` blocks wide, and vectors in
// W.v(0).
template <typename real>
tsk_status cpow_run(const CpowWork& W, int64_t nsteps, bool affine, int band, int doublings,
                    const CpowOut<real>& out, hipStream_t s) {
    const int ld = W.ld, ts = 32 * W.mt, wt = (ld + ts - 1) / ts;
    int b = W.first, vb = 0;
    for (int k = 0; k < doublings; ++k) {
        CpowArgs<real> g{};
        g.A = g.B = W.D<real>(b);
        g.out = W.D<real>(b ^ 1);
        g.vin = W.v<real>(vb);
        g.vout = W.v<real>(vb ^ 1);
        g.ld = ld;
        g.count = W.count;
        g.band_a = g.band_b = band;
        g.band_c = 2 * band;
        g.tile_blocks = wt * wt;
        g.bit = int((nsteps >> k) & 1);
        g.affine = affine ? 1 : 0;
        const int vblocks = (g.bit || g.affine) ? ld / 4 : 0;
        const dim3 grid(unsigned((g.tile_blocks + vblocks) * W.count));
        cpow_gemm<real, CPOW_SQUARE>(W, grid, g, s);
        b ^= 1;
        if (vblocks) vb ^= 1;
        band = std::min(2 * band, ld);
    }
    for (int64_t r = nsteps >> doublings; r > 0; --r) {
        CpowArgs<real> g{};
        g.A = W.D<real>(b);
        g.vin = W.v<real>(vb);
        g.vout = W.v<real>(vb ^ 1);
        g.ld = ld;
        g.count = W.count;
        g.band_a = band;
        g.ts = 16 * W.mt;
        g.affine = affine ? 1 : 0;
        hipLaunchKernelGGL(k_cpow_apply<real>, dim3(unsigned(ld / 4 * W.count)), dim3(4 * kWave), 0, s, g, out,
                           r == 1 ? 1 : 0);
        vb ^= 1;
    }
    TSK_HIP(hipGetLastError());
    return TSK_OK;
}

}  // namespace tsk
