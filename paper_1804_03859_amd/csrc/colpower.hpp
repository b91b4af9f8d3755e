// Time integration of a one-harmonic parallel base flow by repeated squaring of
// the step (the chains of colcouple.hpp).
//
// One Lawson RK4 step of a chain of n coupled modes is a real n x n matrix S =
// I + D that does not change over the integration, so the nsteps steps of a
// matvec are S^nsteps x.  Stepping takes nsteps dependent RK4 steps of one
// wavefront; the binary expansion of nsteps takes log2(nsteps) squarings of an
// n x n matrix, which run on the matrix cores, and one matrix-vector product
// per set bit:
//     for the bits of nsteps from the lowest: if set, x <- x + D x;  D <- 2 D + D D.
// Where a mode is still near 1, D, not S, is squared: (I + D)^2 - I = 2 D + D D keeps
// the relative accuracy of the small step matrix.  A mode damped to s < 1/2 would
// lose its own in D = s - 1, so its diagonal entry turns to s there: the matrix that
// is kept is C = S - diag(b), b = 1 or 0 by the row, and the recursion
//     x <- b x + C x;  C_ij <- (b_i + b_j) C_ij + (C C)_ij.
// The result is closer to the exact power than the nsteps rounded steps are, in the
// norm (relative error against long double at 128^2, T = 1: 2e-16 instead of 6e-15 in
// FP64, 1.3e-7 instead of 2.7e-6 in FP32) and mode by mode (worst error in units of
// eps max_k |S^(n-k)| |S^k| |x|, 200 steps of a chain at 128^2, 256^2, Re = 20: 12 to 15
// stepped, 2 to 3 here; with b = 1 throughout 3e4 and more, and no digit of a column
// damped below eps).  Nothing is kept between calls: every call forms C from the
// parameters.
//
// Chains c and nh - c of a column hold the modes ky and -ky; with u_i = (-1)^i
// s_{len-1-i} the second obeys the first's equations, so one workgroup squares
// one matrix for both and applies it to four real vectors.
//
// Layout.  A workgroup holds C in LDS, row pitch NP + 4 (the fragment reads of 16
// rows x 4 columns then touch each bank equally often), and squares it in place:
// the C tiles of 16 x 16 are accumulated in registers by
// v_mfma_{f64,f32}_16x16x4 starting from (b_i + b_j) C and written after a barrier.  One
// wavefront owns a row of tiles, so an A fragment is read once for the whole
// row; chains of two tiles take four wavefronts of one tile (the shortest
// dependent chain), chains of one tile a single wavefront and no barrier.  S has
// half-bandwidth 4 and S^(2^k) 4 2^k, so the first three squarings of chains of
// four and more tiles run on the five tiles next to the diagonal.
//
// Bound: the matrix cores (64 cycles per FP64 and 32 per FP32 16x16x4 product and
// SIMD) once the launch fills the device, the chain of dependent squarings below.
#pragma once

#include "colcouple.hpp"

namespace tsk {

constexpr int kPowMaxTiles = 6;  // chains of up to 96 modes
// Wavefronts of a workgroup for chains of tc tiles.
__host__ __device__ constexpr int power_waves(int tc) { return tc == 1 ? 1 : tc == 2 ? 4 : tc; }

template <typename real> struct MfmaTile;
template <> struct MfmaTile<double> {
    using V = double __attribute__((ext_vector_type(4)));
    static __device__ inline V fma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct MfmaTile<float> {
    using V = float __attribute__((ext_vector_type(4)));
    static __device__ inline V fma(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Chain pairs (c, nh - c), c = 0 .. nh / 2, of every column, and the kx = 0 column.
__host__ __device__ inline int power_blocks(int M, int nh) { return 1 + M * (nh / 2 + 1); }
__host__ __device__ inline int power_tiles(int M, int nh) { return ((2 * M + 1 + nh - 1) / nh + 15) / 16; }
template <typename real, int TC> constexpr int power_lds_bytes() {
    constexpr int NP = 16 * TC;
    return int(sizeof(real)) * (NP * (NP + 4) + 2 * NP * 4 + NP) + 8 * 4 * (NP + 8);
}

// Squarings k before the matrix D of 2^k steps is applied nsteps >> k times: one
// more squaring has to save more products than it costs.  Measured costs of a
// squaring / a product at 128^2, 256^2, 384^2, 512^2 (2, 3, 4, 6 tiles), FP64: 0.6 /
// 0.33, 1.5 / 0.47, 4.3 / 0.7 and 18 / 1.6 us (FP32 0.33 / 0.24 to 9 / 0.7).
template <int TC> __device__ inline int power_squarings(int nsteps) {
    constexpr int ratio = TC <= 2 ? 1 : TC == 3 ? 3 : TC == 4 ? 5 : 7;
    int k = 0;
    while ((nsteps >> k) - (nsteps >> (k + 1)) > ratio) ++k;
    return k;
}
template <int TC> __device__ inline int clamp_tile(int t) { return t < 0 ? 0 : t < TC ? t : TC - 1; }

// One chain pair (slot of power_blocks) of instance I, chains of up to TC tiles.
// ADJ: the transposed propagator ((S^T)^nsteps; the y-origin phases stay where
// they are).  Wavefronts beyond power_waves(TC) must not enter.
template <typename real, int TC, bool ADJ>
__device__ __forceinline__ void couple_power(const ColInst<real>& I, int jstep, int slot, char* lds_power) {
    using T = MfmaTile<real>;
    using V = typename T::V;
    constexpr int NP = 16 * TC, P = NP + 4, NT = power_waves(TC) * kWave;
    constexpr int NJ = TC == 2 ? 1 : TC;      // tiles of a wavefront
    constexpr int PR = TC == 2 ? 8 : 4;       // threads per row of a matrix-vector product
    static_assert(NP * PR <= NT, "one row per PR threads");
    const int M = I.M, nh = I.nh;
    const int tid = int(threadIdx.x), lane = tid % kWave, wv = tid / kWave;
    const real* __restrict__ xin = I.xbase + jstep * I.xstride;
    real* __restrict__ yout = I.y;
    const double alpha = I.alpha, Re = I.Re, dt = I.dt;
    if (slot == 0) {  // kx = 0: the integrating factor alone
        for (int q = tid; q < M; q += NT) {
            const double jy = q + 1, E = exp(-jy * jy * dt / Re * I.nsteps);
            yout[2 * q] = real(E * double(xin[2 * q]));
            yout[2 * q + 1] = real(E * double(xin[2 * q + 1]));
        }
        return;
    }
    double* sG = reinterpret_cast<double*>(lds_power);  // factors of the modes, 4 zeros at either end
    double* sE = sG + (NP + 8);                         // Eh
    double* s1 = sE + (NP + 8);                         // E1
    double* sF = s1 + (NP + 8);                         // E1 - b
    real* D = reinterpret_cast<real*>(sF + (NP + 8));
    real* vec = D + NP * P;       // [2][NP][4]
    real* sB = vec + 2 * NP * 4;  // b
    const int pr = nh / 2 + 1, kx = 1 + (slot - 1) / pr, c = (slot - 1) % pr;
    const double kxv = alpha * kx;
    const int jy0 = -M + ((c + M) % nh), len = (M - jy0) / nh + 1;
    const bool two = (nh - c) % nh != c;  // the mirrored chain is another one
    const int NM = 2 * M + 1;
    const int64_t seg = 2ll * M + int64_t(kx - 1) * 2 * NM;
    const real* xs = xin + seg;
    real* ys = yout + seg;

    for (int i = tid; i < NP + 8; i += NT) {
        const int t = i - 4;
        double g = 0.0, eh = 0.0, e1 = 0.0, e1b = 0.0;
        bool near1 = true;
        if (t >= 0 && t < len) {
            const double jy = jy0 + nh * t, K2 = kxv * kxv + jy * jy;
            g = 0.5 * I.amp * kxv * (1.0 - I.cprop / K2);
            const double q = -K2 * (0.5 * dt) / Re, ehm = expm1(q);
            eh = ehm > -0.5 ? 1.0 + ehm : exp(q);
            const double e1m = ehm * (2.0 + ehm);
            near1 = e1m > -0.5;
            e1 = near1 ? 1.0 + e1m : eh * eh;
            e1b = near1 ? e1m : e1;
        }
        sG[i] = g;
        sE[i] = eh;
        s1[i] = e1;
        sF[i] = e1b;
        if (t >= 0 && t < NP) sB[t] = near1 ? real(1) : real(0);
    }
    for (int i = tid; i < NP * P; i += NT) D[i] = real(0);
    // columns of the vector block: (re, im) of the chain, (re, im) of the mirrored one
    double ph_c = 1.0, ph_s = 0.0;  // e^{i ky y0} of this thread's mode (-ky: its conjugate)
    if (tid < NP) {
        real v[4] = {real(0), real(0), real(0), real(0)};
        if (tid < len) {
            const int jy = jy0 + nh * tid;
            if (I.y0 != 0.0) sincos(double(jy) * I.y0, &ph_s, &ph_c);
            const real pc = real(ph_c), ps = real(ph_s);
            const real a = xs[2 * (jy + M)], b = xs[2 * (jy + M) + 1];
            v[0] = a * pc - b * ps;
            v[1] = a * ps + b * pc;
            if (two) {
                const real ma = xs[2 * (M - jy)], mb = xs[2 * (M - jy) + 1], sg = tid & 1 ? real(-1) : real(1);
                v[2] = sg * (ma * pc + mb * ps);
                v[3] = sg * (mb * pc - ma * ps);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) vec[tid * 4 + q] = v[q];
    }
    __syncthreads();
    if (tid < len) {
        // column tid of C: the RK4 step of a unit vector, nonzero at offsets -4..4
        double g[11], eh[9], e1[9];
#pragma unroll
        for (int o = 0; o < 9; ++o) {
            g[o + 1] = sG[tid + o];
            eh[o] = sE[tid + o];
            e1[o] = s1[tid + o];
        }
        g[0] = g[10] = 0.0;
        double s[11], k1[9], sum[9];
#pragma unroll
        for (int o = 0; o < 11; ++o) s[o] = o == 5 ? 1.0 : 0.0;
        auto advect = [&](double (&n)[9]) {
#pragma unroll
            for (int o = 0; o < 9; ++o) n[o] = g[o + 2] * s[o + 2] - g[o] * s[o];
        };
        const double h = dt, h2 = 0.5 * dt;
        advect(k1);
#pragma unroll
        for (int o = 0; o < 9; ++o) sum[o] = e1[o] * k1[o];
#pragma unroll
        for (int o = 0; o < 9; ++o) s[o + 1] = eh[o] * ((o == 4 ? 1.0 : 0.0) + h2 * k1[o]);
        advect(k1);
#pragma unroll
        for (int o = 0; o < 9; ++o) sum[o] += 2.0 * eh[o] * k1[o];
#pragma unroll
        for (int o = 0; o < 9; ++o) s[o + 1] = (o == 4 ? eh[o] : 0.0) + h2 * k1[o];
        advect(k1);
#pragma unroll
        for (int o = 0; o < 9; ++o) sum[o] += 2.0 * eh[o] * k1[o];
#pragma unroll
        for (int o = 0; o < 9; ++o) s[o + 1] = (o == 4 ? e1[o] : 0.0) + h * eh[o] * k1[o];
        advect(k1);
        const double h6 = dt / 6.0;
#pragma unroll
        for (int o = 0; o < 9; ++o) {
            const int t = tid + o - 4;
            const double d = (o == 4 ? sF[tid + 4] : 0.0) + h6 * (sum[o] + k1[o]);
            if (t >= 0 && t < len) D[ADJ ? tid * P + t : t * P + tid] = real(d);
        }
    }
    __syncthreads();

    const int ti = TC == 2 ? wv >> 1 : wv, tj0 = TC == 2 ? wv & 1 : 0;
    const real* pa = D + (16 * ti + (lane & 15)) * P + (lane >> 4);  // A fragments of the row of tiles
    const real* pb = D + (lane >> 4) * P + (lane & 15);              // B fragments of tile (0, 0)
    real* pc = D + 16 * ti * P + (lane & 15);                        // C tile (ti, 0), row offsets T::row
    const int row = tid / PR, sgm = tid % PR;  // of a matrix-vector product
    int cur = 0, bw = 4;
    unsigned e = unsigned(I.nsteps);
    for (int left = power_squarings<TC>(I.nsteps); left > 0; --left) {
        if (e & 1u) {  // x <- b x + C x, PR threads per row
            const real* vc = vec + cur * NP * 4;
            const real b = row < NP ? sB[row] : real(0);
            real a[4] = {real(0), real(0), real(0), real(0)};
            if (row < len) {
                const int lo = row > bw ? (row - bw) / PR * PR : 0, hi = row + bw + 1 < len ? row + bw + 1 : len;
                for (int k = lo + sgm; k < hi; k += PR) {
                    const real d = D[row * P + k];
#pragma unroll
                    for (int q = 0; q < 4; ++q) a[q] = fma(d, vc[k * 4 + q], a[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] += xor_lane<1>(a[q], lane);
                a[q] += xor_lane<2>(a[q], lane);
                if constexpr (PR >= 8) a[q] += xor_lane<4>(a[q], lane);
            }
            if (sgm == 0 && row < NP)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    vec[(cur ^ 1) * NP * 4 + row * 4 + q] = fma(b, vc[row * 4 + q], a[q]);
            cur ^= 1;
        }
        e >>= 1;
        // b of the rows of the tiles; of the lane's diagonal entry b and whether it turns from
        // s - 1 to s (judged by the square it is about to become, so off the products' path)
        real br[4], one[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) br[r] = sB[16 * ti + T::row(lane, r)];
        const real bd = sB[16 * ti + (lane & 15)], sd = real(1) + D[(16 * ti + (lane & 15)) * (P + 1)];
        const bool turn = bd != real(0) && sd * sd < real(0.5);
#pragma unroll
        for (int r = 0; r < 4; ++r) one[r] = turn && T::row(lane, r) == (lane & 15) ? real(1) : real(0);
        if (TC >= 4 && bw <= 16) {
            // C tiles ti - 2 .. ti + 2 from A and B tiles next to the diagonal; tiles
            // outside the matrix are read clamped, A as zero, and not written
            V acc[5];
#pragma unroll
            for (int d = 0; d < 5; ++d) {
                const int tj = clamp_tile<TC>(ti + d - 2);
                const real bc = sB[16 * tj + (lane & 15)];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[d][r] = fma(br[r] + bc, pc[T::row(lane, r) * P + 16 * tj], d == 2 ? one[r] : real(0));
            }
#pragma unroll
            for (int dk = -1; dk <= 1; ++dk) {
                const int tk = clamp_tile<TC>(ti + dk);
                real a[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = tk == ti + dk ? pa[16 * tk + 4 * q] : real(0);
#pragma unroll
                for (int dj = -1; dj <= 1; ++dj) {
                    const int tj = clamp_tile<TC>(tk + dj);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[dk + dj + 2] = T::fma(a[q], pb[(16 * tk + 4 * q) * P + 16 * tj], acc[dk + dj + 2]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int d = 0; d < 5; ++d) {
                const int tj = ti + d - 2;
                if (tj >= 0 && tj < TC)
#pragma unroll
                    for (int r = 0; r < 4; ++r) pc[T::row(lane, r) * P + 16 * tj] = acc[d][r];
            }
        } else {
            V acc[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const real bc = sB[16 * (tj0 + j) + (lane & 15)];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[j][r] = fma(br[r] + bc, pc[T::row(lane, r) * P + 16 * (tj0 + j)],
                                    tj0 + j == ti ? one[r] : real(0));
            }
#pragma unroll
            for (int tk = 0; tk < TC; ++tk) {
                real a[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = pa[16 * tk + 4 * q];
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[j] = T::fma(a[q], pb[(16 * tk + 4 * q) * P + 16 * (tj0 + j)], acc[j]);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) pc[T::row(lane, r) * P + 16 * (tj0 + j)] = acc[j][r];
        }
        if (turn && lane < 16) sB[16 * ti + lane] = real(0);
        __syncthreads();
        bw = 2 * bw < len ? 2 * bw : len;
    }
    // the e remaining applications of the last C, its rows in registers
    constexpr int NR = NP / PR;
    real dr[NR];
    const real bo = row < NP ? sB[row] : real(0);
#pragma unroll
    for (int i = 0; i < NR; ++i) dr[i] = row < NP ? D[row * P + sgm + PR * i] : real(0);
    for (; e > 0; --e) {
        const real* vc = vec + cur * NP * 4;
        real a[4] = {real(0), real(0), real(0), real(0)};
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = fma(dr[i], vc[(sgm + PR * i) * 4 + q], a[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] += xor_lane<1>(a[q], lane);
            a[q] += xor_lane<2>(a[q], lane);
            if constexpr (PR >= 8) a[q] += xor_lane<4>(a[q], lane);
        }
        cur ^= 1;
        if (sgm == 0 && row < NP)
#pragma unroll
            for (int q = 0; q < 4; ++q) vec[cur * NP * 4 + row * 4 + q] = fma(bo, vc[row * 4 + q], a[q]);
        __syncthreads();
    }
    if (tid < len) {
        const int jy = jy0 + nh * tid;
        const real pc = real(ph_c), ps = real(ph_s);
        const real* v = vec + cur * NP * 4 + tid * 4;
        ys[2 * (jy + M)] = v[0] * pc + v[1] * ps;
        ys[2 * (jy + M) + 1] = v[1] * pc - v[0] * ps;
        if (two) {
            const real sg = tid & 1 ? real(-1) : real(1), a = sg * v[2], b = sg * v[3];
            ys[2 * (M - jy)] = a * pc - b * ps;
            ys[2 * (M - jy) + 1] = b * pc + a * ps;
        }
    }
}

// One instance.  Grid x: power_blocks.  (Three wavefronts per SIMD are what the LDS of
// four and five tiles lets in.)
template <typename real, int TC, bool ADJ>
__global__ __launch_bounds__(power_waves(TC) * kWave, TC == 6 ? 2 : 3) void k_couple_power(ColInst<real> I) {
    extern __shared__ __align__(16) char lds_power[];
    stepper_wave_priority();
    couple_power<real, TC, ADJ>(I, 0, int(blockIdx.x), lds_power);
}

// Batch: grid x = power_blocks of the largest instance, grid y and the instance
// table as in k_colstep_couple; every instance runs the code of its own tile
// count (the same arithmetic as alone), the workgroup sized for the largest.
template <typename real>
__global__ __launch_bounds__(kPowMaxTiles * kWave, 4) void k_couple_power_batch(const ColInst<real>* __restrict__ insts,
                                                                             const int* __restrict__ ids, int jstep) {
    extern __shared__ __align__(16) char lds_power[];
    stepper_wave_priority();
    const ColInst<real>& I = insts[ids[blockIdx.y]];
    if ((I.active && *I.active == 0) || jstep >= I.jmax) return;
    const int tc = power_tiles(I.M, I.nh), slot = int(blockIdx.x);
    if (slot >= power_blocks(I.M, I.nh) || int(threadIdx.x) >= power_waves(tc) * kWave) return;
    switch (tc) {
        case 1: return couple_power<real, 1, false>(I, jstep, slot, lds_power);
        case 2: return couple_power<real, 2, false>(I, jstep, slot, lds_power);
        case 3: return couple_power<real, 3, false>(I, jstep, slot, lds_power);
        case 4: return couple_power<real, 4, false>(I, jstep, slot, lds_power);
        case 5: return couple_power<real, 5, false>(I, jstep, slot, lds_power);
        default: return couple_power<real, 6, false>(I, jstep, slot, lds_power);
    }
}

}  // namespace tsk
