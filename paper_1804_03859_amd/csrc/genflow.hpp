// The pipeline of kolmo2d.hip in one launch per integration: the column and row
// workgroups stay resident and pass the fields between them directly.
//
// Two launches per stage cost about 2.4 us each before any work, and every launch
// loads the twiddles, the state and the base fields again and evaluates its
// exponentials.  Here the MC column workgroups and N / 2 row workgroups each keep
// theirs in registers and LDS for all stages; a stage is two hops between them.
// Measured, us per hop (launches / this): FP64 16^2 4.0 / 1.4, 96^2 4.8 / 2.9, 128^2 5.3 /
// 3.1, 256^2 6.5 / 5.3; FP32 16^2 3.8 / 1.2, 256^2 5.5 / 3.4.  A hop is about 1 us of memory latency, two
// transforms by one wavefront (fft.hpp's register form; through LDS with workgroup
// barriers a hop took 2.1, 3.9, 4.2, 7.1 and 4.2) and, from 192^2 in FP64 on, the traffic
// of the words.
//
// Exchange.  A hop carries 32-bit halves of the values in 64-bit words (tag << 32 |
// bits), the tag numbering the stage.  They are written and read two at a time by
// 16-byte buffer accesses of device scope.  What is assumed of these: an aligned
// 8-byte word is seen whole (a lane's aligned 16 bytes are one request to one cache
// line); nothing is assumed of the order of words, not even within an access.  A
// consumer polls the words themselves until they carry its tag: one trip through
// memory, no flags, no fences.  No word is overwritten before it was read: its producer writes the next stage
// only after it has received words that its consumers computed from this one.  Tags
// count on from call to call (a graph replays its own range: the words then hold the
// last tag of some range, never the first one of this).
//
// Waits are bounded.  The workgroups need not all be resident for correctness: a
// wavefront that waits kFlowPolls polls in vain (workgroups held back by other
// work on the GPU) sets `failed` and stops waiting, as do all others then, so that
// the launch drains; k_flow_repair, launched behind it, computes the integration by
// one workgroup with plain memory if it finds `failed` set, and clears the words.
// That takes the 0.1 s of the wait and 13 (64^2) to 62 (256^2) times as long as the stage
// launches, 3.5 ms a step at 256^2 FP64, so it also notes it in host memory: the
// operator's later integrations run stage by stage.  So do all on a device whose CUs
// cannot hold the launch (a partition of the GPU).
//
// A complex value is a cell of 4 (FP64) or 2 (FP32) words, moved as one or two quads of
// 16 bytes (the words of an access need not arrive together).  Layouts (p: row pair,
// r: row of it, q: quad):
//     columns -> rows   [p][field][kx][q][r]   a row wavefront reads runs of kx
//     rows -> columns   [kx][field][p][q][r]   a column wavefront reads runs of y
// so that readers, which poll, touch whole lines, and adjacent lanes of a writer 32 bytes
// at once.
#pragma once

#include "fft.hpp"

namespace tsk {

constexpr int kFlowPolls = 1 << 17;  // about 0.1 s

template <typename real> struct FlowArgs {
    using C = cplx<real>;
    const real* x;
    real* y;
    real *U, *V, *Ox, *Oy;  // base fields
    const real* fvec;       // forcing, or null
    const C* tw;
    unsigned long long* toRows;
    unsigned long long* toCols;
    unsigned* failed;
    unsigned* note;  // host memory, set once a launch has given up (or null)
    unsigned tag;    // of the first stage
    int polls, nsteps;
    double alpha, Re, dt, U0;
};

// ---- cells --------------------------------------------------------------------------
typedef unsigned quad __attribute__((ext_vector_type(4)));  // two words: bits, tag, bits, tag
template <typename real> constexpr int kFlowQuads = sizeof(real) / 4;  // of a cell

// Device-scope accesses past the caches of one XCD (sc1), loads not to be merged or
// moved (the volatile bit).
constexpr int kFlowScope = 1 << 4, kFlowVolatile = int(1u << 31);
using FlowBuf = __amdgpu_buffer_rsrc_t;
__device__ inline FlowBuf flow_buf(unsigned long long* p, size_t words) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, int(words * sizeof(unsigned long long)), 0x00027000);
}

__device__ inline void flow_pack(double2 v, unsigned tag, quad (&d)[2]) {
    const unsigned long long a = __double_as_longlong(v.x), b = __double_as_longlong(v.y);
    d[0] = quad{unsigned(a), tag, unsigned(a >> 32), tag};
    d[1] = quad{unsigned(b), tag, unsigned(b >> 32), tag};
}
__device__ inline void flow_pack(float2 v, unsigned tag, quad (&d)[1]) {
    d[0] = quad{__float_as_uint(v.x), tag, __float_as_uint(v.y), tag};
}
__device__ inline double2 flow_value(const quad (&d)[2]) {
    return make_double2(__longlong_as_double((unsigned long long)(d[0].z) << 32 | d[0].x),
                        __longlong_as_double((unsigned long long)(d[1].z) << 32 | d[1].x));
}
__device__ inline float2 flow_value(const quad (&d)[1]) {
    return make_float2(__uint_as_float(d[0].x), __uint_as_float(d[0].z));
}

// Byte offset of quad i of a cell (cells 2 c and 2 c + 1 are a pair of rows).
template <int Q> __device__ inline int flow_at(unsigned cell, int i) {
    return int((cell >> 1) * (32 * Q) + (cell & 1) * 16 + 32 * i);
}
template <typename C, typename real = decltype(C{}.x)>
__device__ inline void flow_send(FlowBuf buf, unsigned cell, C v, unsigned tag) {
    constexpr int Q = kFlowQuads<real>;
    quad d[Q];
    flow_pack(v, tag, d);
#pragma unroll
    for (int i = 0; i < Q; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(d[i], buf, flow_at<Q>(cell, i), 0, kFlowScope);
}

// K cells per lane into v.  LIGHT: polls one access per lane until it has arrived and
// reads the rest then; else polls everything.  One trip more after the arrival against
// polls that crowd the stores they wait for: us per hop all / light, FP64 96^2 2.96 /
// 3.02, 128^2 3.40 / 3.23, 256^2 6.86 / 5.42; FP32 192^2 2.84 / 2.91, 256^2 3.98 / 3.63;
// light for the four-field direction alone 128^2 3.07, 256^2 5.28, FP32 256^2 3.43.  Two
// polls in flight are no faster.
struct FlowWait {
    unsigned* failed;
    int polls;
    bool dead = false;  // stopped waiting (uniform over the wavefront)
};
template <bool LIGHT, typename C, int K, typename real = decltype(C{}.x)>
__device__ inline void flow_recv(FlowBuf buf, const unsigned (&cell)[K], unsigned tag, C (&v)[K], FlowWait& wt) {
    constexpr int Q = kFlowQuads<real>;
    quad d[K][Q];
    bool all = !LIGHT;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < Q; ++i) d[k][i] = quad{0, 0, 0, 0};
    for (int n = 0; !wt.dead; ++n) {
        bool ok = true;
        if (all) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    d[k][i] = __builtin_amdgcn_raw_buffer_load_b128(buf, flow_at<Q>(cell[k], i), 0,
                                                                    kFlowScope | kFlowVolatile);
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i) ok = ok && d[k][i].y == tag && d[k][i].w == tag;
            if (__all(ok)) break;
        } else {
            const quad t = __builtin_amdgcn_raw_buffer_load_b128(buf, flow_at<Q>(cell[K - 1], Q - 1), 0,
                                                                 kFlowScope | kFlowVolatile);
            all = __all(t.y == tag);
        }
        if (n >= wt.polls) {
            __hip_atomic_store(wt.failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wt.dead = true;
        } else if ((n & 63) == 63) {
            wt.dead = __builtin_amdgcn_readfirstlane(
                          __hip_atomic_load(wt.failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = flow_value(d[k]);
}

// ---- geometry -----------------------------------------------------------------------
template <typename real, int N> struct FlowGeo {
    static constexpr int M = (N - 1) / 3, MC = M + 1, NM = 2 * M + 1;
    static constexpr int KI = (MC + kWave - 1) / kWave;      // kx per lane
    static constexpr int SI = (2 * MC + kWave - 1) / kWave;  // (kx, row of the pair) per lane
    static constexpr int blocks = MC + N / 2;
    static constexpr size_t words(int fields) { return size_t(fields) * 2 * kFlowQuads<real> * MC * N; }
    // Cells.
    static __device__ inline unsigned row_at(int fields, int f, int y, int kx) {
        return unsigned((((y >> 1) * fields + f) * MC + kx) * 2 + (y & 1));
    }
    static __device__ inline unsigned col_at(int fields, int f, int kx, int y) {
        return unsigned((kx * fields + f) * N + y);
    }
    // flow_recv's light polls: readers of four fields, from 1 KB a transform on.
    static constexpr bool light(int fields) { return fields == 4 && N * sizeof(real) >= 1024; }
};

// Grids that run this way: one mode per thread, and workgroups small enough that the
// CUs hold four launches at once.  Beyond (384^2, 512^2) a launch per stage kernel.
constexpr bool flow_fits(int N) { return N <= 256; }
constexpr int kFlowSteps = 512;  // steps per launch (a few ms)

// FP64 at N = 256: 35 KB and at most 128 registers, four workgroups per CU, so that four
// launches (one per hardware queue of a process) are resident together.
template <typename real, int N> struct FlowLds {
    cplx<real> A[4][N], B[4][N], S[FlowGeo<real, N>::NM];
};

// A packed mode of a column by its grid index t, or none: entry of the segment,
// conjugated (kx = 0) or not.
template <int M> __device__ inline bool flow_mode(int t, int N, int kx, int& e, bool& conj, int& jy) {
    jy = 2 * t <= N ? t : t - N;
    conj = kx == 0 && jy < 0;
    if (conj) jy = -jy;
    e = kx == 0 ? jy - 1 : jy + M;
    return jy <= M && jy >= -M && (kx > 0 || jy > 0);
}

// The pair's half spectra (kx = 0 .. M of rows 0 and 1 at src) received into the spectrum
// of row 0 + i row 1 (its modes beyond M stay zero).
template <typename real, int N, int F, int K, typename C = cplx<real>>
__device__ inline void flow_unpair(FlowBuf rows, const unsigned (&src)[K], unsigned tag, FlowWait& wt, C* a,
                                   int lane) {
    using G = FlowGeo<real, N>;
    C v[K];
    flow_recv<G::light(F)>(rows, src, tag, v, wt);
#pragma unroll
    for (int i = 0; i < K / 2; ++i) {
        const int k = lane + kWave * i;
        if (k > G::M) continue;
        C g0 = v[2 * i], g1 = v[2 * i + 1];
        if (k == 0) {  // the kx = 0 column of a real field is real
            g0.y = real(0);
            g1.y = real(0);
        }
        a[k] = cmk<C>(g0.x - g1.y, g0.y + g1.x);
        if (k > 0) a[N - k] = cmk<C>(g0.x + g1.y, g1.x - g0.y);
    }
    wave_lds_sync();
}
// The spectrum of row 0 + i row 1 (k = l + L r, through Z) split into the pair's half
// spectra and sent as field f.
template <typename real, int N, typename C = cplx<real>>
__device__ inline void flow_split(FlowBuf cols, const LaneFft<real, N>& ft, const C (&v)[LaneFft<real, N>::R], C* Z,
                                  int fields, int f, int y0, unsigned tag, int lane) {
    using G = FlowGeo<real, N>;
    using T = LaneFft<real, N>;
#pragma unroll
    for (int r = 0; r < T::R; ++r)
        if (lane < T::L) Z[lane + T::L * r] = v[r];
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < G::SI; ++i) {
        const int k = (lane + kWave * i) >> 1;
        if (k > G::M) continue;
        const C za = Z[k], zb = cconj(Z[k == 0 ? 0 : N - k]);
        const C h = (lane & 1) == 0 ? cmk<C>(real(0.5) * (za.x + zb.x), real(0.5) * (za.y + zb.y))
                                    : cmk<C>(real(0.5) * (za.y - zb.y), real(-0.5) * (za.x - zb.x));
        flow_send(cols, G::col_at(fields, f, k, y0 + (lane & 1)), h, tag);
    }
    wave_lds_sync();
}

// The barriers below: column workgroups put their stage input into S (barrier), its
// transforms go out; the answer's transform goes to A (barrier).  A row workgroup's
// wavefronts put their transforms into B (one barrier); they write B again only on
// words that the columns send after all of this workgroup's.

// ---- forward: linearized (ROW_LIN) and nonlinear (ROW_NL) ----------------------------
template <typename real, int N>
__device__ void flow_col(const FlowArgs<real>& g, FlowLds<real, N>& s, int kx) {
    using C = cplx<real>;
    using G = FlowGeo<real, N>;
    using T = LaneFft<real, N>;
    constexpr int M = G::M, NM = G::NM, R = T::R, L = T::L;
    const int tid = int(threadIdx.x), lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int nq = kx == 0 ? M : NM;
    const int64_t o = (kx == 0 ? 0 : 2ll * M + int64_t(kx - 1) * 2 * NM) + 2 * tid;
    const double kxv = g.alpha * kx;
    FlowWait wt{g.failed, g.polls};
    const FlowBuf rows = flow_buf(g.toRows, G::words(4)), cols = flow_buf(g.toCols, G::words(1));
    T ft;
    ft.init(g.tw);
    // the thread's mode
    const bool act = tid < nq;
    const int my = kx == 0 ? tid + 1 : tid - M, ix = my < 0 ? my + N : my;
    double e1 = 0.0, eh = 0.0, fx = 0.0, fy = 0.0;
    real wx = 0, wy = 0, ax = 0, ay = 0;
    if (act) {
        const double K2 = kxv * kxv + double(my) * my;
        e1 = exp(-K2 * g.dt / g.Re);
        eh = exp(-K2 * (0.5 * g.dt) / g.Re);
        wx = g.x[o];
        wy = g.x[o + 1];
        if (g.fvec) {
            fx = double(g.fvec[o]);
            fy = double(g.fvec[o + 1]);
        }
        s.S[tid] = cmk<C>(wx, wy);
    }
    // wavefront f: factors of derived field f (i c s; c = kx, ky, ky/K^2, -kx/K^2) at the
    // lane's points of the inverse transform
    int en[R];
    unsigned keep = 0, conjs = 0;
    double cf[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int e, jy;
        bool conj;
        const bool kept = flow_mode<M>(r + R * ft.rev, N, kx, e, conj, jy);
        const double K2 = kept ? kxv * kxv + double(jy) * jy : 1.0;
        cf[r] = wv == 0 ? kxv : wv == 1 ? double(jy) : wv == 2 ? double(jy) / K2 : -kxv / K2;
        en[r] = kept ? e : 0;
        keep |= unsigned(kept) << r;
        conjs |= unsigned(conj) << r;
    }
    const double h = g.dt, h2 = 0.5 * g.dt, h3 = g.dt / 3.0, h6 = g.dt / 6.0;
    const double scl = -1.0 / (double(N) * N);
    unsigned tag = g.tag;
    for (int st = 0; st < g.nsteps; ++st)
        for (int q = 0; q < 4; ++q, ++tag) {
            __syncthreads();
            C v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const C sv = s.S[en[r]];
                const real dx = real(-cf[r] * double(sv.y)), dy = real(cf[r] * double(sv.x));
                const bool kept = keep >> r & 1;
                v[r] = cmk<C>(kept ? dx : real(0), kept ? ((conjs >> r & 1) ? -dy : dy) : real(0));
            }
            ft.template dit<+1>(v);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane < L) flow_send(rows, G::row_at(4, wv, lane + L * r, kx), v[r], tag);
            if (wv == 0) {
                unsigned p[R];
#pragma unroll
                for (int r = 0; r < R; ++r) p[r] = G::col_at(1, 0, kx, ft.l + L * r);
                flow_recv<G::light(1)>(cols, p, tag, v, wt);
                ft.template dif<-1>(v);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (lane < L) s.A[0][r + R * ft.rev] = v[r];
            }
            __syncthreads();
            if (act) {
                const C xr = s.A[0][ix];
                const double nx = scl * double(xr.x) + fx, ny = scl * double(xr.y) + fy;
                double sx, sy;
                if (q == 0) {
                    ax = real(e1 * (double(wx) + h6 * nx));
                    ay = real(e1 * (double(wy) + h6 * ny));
                    sx = eh * (double(wx) + h2 * nx);
                    sy = eh * (double(wy) + h2 * ny);
                } else if (q == 3) {
                    wx = real(double(ax) + h6 * nx);
                    wy = real(double(ay) + h6 * ny);
                    sx = double(wx);
                    sy = double(wy);
                } else {
                    ax = real(double(ax) + h3 * eh * nx);
                    ay = real(double(ay) + h3 * eh * ny);
                    sx = q == 1 ? eh * double(wx) + h2 * nx : e1 * double(wx) + h * eh * nx;
                    sy = q == 1 ? eh * double(wy) + h2 * ny : e1 * double(wy) + h * eh * ny;
                }
                s.S[tid] = cmk<C>(real(sx), real(sy));
            }
        }
    if (act) {
        g.y[o] = wx;
        g.y[o + 1] = wy;
    }
}

// The base field that multiplies field f (wavefront f's, d_x w, d_y w, u, v) at the lane's
// points x = r + R b(l) of both rows.
template <typename real, int N, int R>
__device__ inline void flow_base(const FlowArgs<real>& g, const LaneFft<real, N>& ft, int f, int y0, real (&b)[R][2]) {
    const real* bf = f == 0 ? g.U : f == 1 ? g.V : f == 2 ? g.Ox : g.Oy;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int r = 0; r < 2; ++r) b[i][r] = bf[size_t(y0 + r) * N + i + R * ft.rev];
}

// Wavefront f transforms field f of both rows of the pair, packed as row 0 + i row 1 (and
// multiplies it by its base field); the first forms the products, or adds them, and
// transforms them back.
template <typename real, int N, bool NL>
__device__ void flow_row(const FlowArgs<real>& g, FlowLds<real, N>& s, int p) {
    using C = cplx<real>;
    using G = FlowGeo<real, N>;
    using T = LaneFft<real, N>;
    constexpr int M = G::M, MC = G::MC, KI = G::KI, R = T::R, L = T::L;
    const int tid = int(threadIdx.x), lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave), y0 = 2 * p;
    FlowWait wt{g.failed, g.polls};
    const FlowBuf rows = flow_buf(g.toRows, G::words(4)), cols = flow_buf(g.toCols, G::words(1));
    T ft;
    ft.init(g.tw);
    real b[R][2];
    if constexpr (!NL) flow_base(g, ft, wv, y0, b);
    unsigned src[2 * KI];
#pragma unroll
    for (int i = 0; i < 2 * KI; ++i) {
        const int k = lane + kWave * (i >> 1);
        src[i] = G::row_at(4, wv, y0 + (i & 1), k <= M ? k : M);
    }
    for (int t = MC + lane; t < N - M; t += kWave) s.A[wv][t] = cmk<C>(real(0), real(0));
    unsigned tag = g.tag;
    for (int n = 0; n < 4 * g.nsteps; ++n, ++tag) {
        flow_unpair<real, N, 4>(rows, src, tag, wt, s.A[wv], lane);
        C v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = s.A[wv][ft.l + L * r];
        ft.template dif<+1>(v);
        if constexpr (!NL) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = cmk<C>(b[r][0] * v[r].x, b[r][1] * v[r].y);
        }
        if (wv > 0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane < L) s.B[wv][lane + L * r] = v[r];
        }
        __syncthreads();
        if (wv > 0) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const C wx = v[r], wy = s.B[1][ft.l + L * r], u = s.B[2][ft.l + L * r], w = s.B[3][ft.l + L * r];
            if constexpr (NL) {
                const real is2 = real(0.70710678118654752440), u0 = real(g.U0);  // the packing factor sqrt(2) once
                v[r] = cmk<C>(is2 * (u.x * wx.x + w.x * wy.x) + u0 * wx.x, is2 * (u.y * wx.y + w.y * wy.y) + u0 * wx.y);
            } else {
                v[r] = cmk<C>(((wx.x + wy.x) + u.x) + w.x, ((wx.y + wy.y) + u.y) + w.y);
            }
        }
        ft.template dit<-1>(v);
        flow_split<real, N>(cols, ft, v, s.B[0], 1, 0, y0, tag, lane);
    }
}

template <typename real, int N, bool NL>
__global__ __launch_bounds__(4 * kWave, 4) void k_flow(FlowArgs<real> g) {
    __shared__ FlowLds<real, N> s;
    const int b = int(blockIdx.x);
    if (b < FlowGeo<real, N>::MC)
        flow_col<real, N>(g, s, b);
    else
        flow_row<real, N, NL>(g, s, b - FlowGeo<real, N>::MC);
}

// ---- the transposed pipeline ----------------------------------------------------------
template <typename real, int N>
__device__ void flow_col_adj(const FlowArgs<real>& g, FlowLds<real, N>& s, int kx) {
    using C = cplx<real>;
    using G = FlowGeo<real, N>;
    using T = LaneFft<real, N>;
    constexpr int M = G::M, NM = G::NM, R = T::R, L = T::L;
    const int tid = int(threadIdx.x), lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int nq = kx == 0 ? M : NM;
    const int64_t o = (kx == 0 ? 0 : 2ll * M + int64_t(kx - 1) * 2 * NM) + 2 * tid;
    const double kxv = g.alpha * kx;
    const double h = g.dt, h2 = 0.5 * g.dt, h3 = g.dt / 3.0, h6 = g.dt / 6.0;
    const double scl = 1.0 / (double(N) * N);
    FlowWait wt{g.failed, g.polls};
    const FlowBuf rows = flow_buf(g.toRows, G::words(1)), cols = flow_buf(g.toCols, G::words(4));
    T ft;
    ft.init(g.tw);
    const bool act = tid < nq;
    const int my = kx == 0 ? tid + 1 : tid - M, ix = my < 0 ? my + N : my;
    double e1 = 0.0, eh = 0.0, cf[4] = {0.0, 0.0, 0.0, 0.0};
    real zx = 0, zy = 0, ax = 0, ay = 0;
    if (act) {
        const double K2 = kxv * kxv + double(my) * my;
        e1 = exp(-K2 * g.dt / g.Re);
        eh = exp(-K2 * (0.5 * g.dt) / g.Re);
        cf[0] = kxv;
        cf[1] = double(my);
        cf[2] = double(my) / K2;
        cf[3] = -kxv / K2;
        zx = g.x[o];
        zy = g.x[o + 1];
        s.S[tid] = cmk<C>(real(h6 * double(zx)), real(h6 * double(zy)));
    }
    int en[R];
    unsigned keep = 0, conjs = 0, src[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int e, jy;
        bool conj;
        const bool kept = flow_mode<M>(r + R * ft.rev, N, kx, e, conj, jy);
        en[r] = kept ? e : 0;
        keep |= unsigned(kept) << r;
        conjs |= unsigned(conj) << r;
        src[r] = G::col_at(4, wv, kx, ft.l + L * r);
    }
    unsigned tag = g.tag;
    for (int st = 0; st < g.nsteps; ++st)
        for (int q = 0; q < 4; ++q, ++tag) {
            __syncthreads();
            C v[R];
            if (wv == 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const C sv = s.S[en[r]];
                    const bool kept = keep >> r & 1;
                    v[r] = cmk<C>(kept ? sv.x : real(0), kept ? ((conjs >> r & 1) ? -sv.y : sv.y) : real(0));
                }
                ft.template dit<+1>(v);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (lane < L) flow_send(rows, G::row_at(1, 0, lane + L * r, kx), v[r], tag);
            }
            flow_recv<G::light(4)>(cols, src, tag, v, wt);
            ft.template dif<-1>(v);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane < L) s.A[wv][r + R * ft.rev] = v[r];
            __syncthreads();
            if (act) {
                double sx = 0.0, sy = 0.0;
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    const C xf = s.A[f][ix];
                    sx -= cf[f] * double(xf.y);
                    sy += cf[f] * double(xf.x);
                }
                sx *= scl;
                sy *= scl;
                double vx, vy;
                if (q == 0) {
                    ax = real(e1 * (double(zx) + sx));
                    ay = real(e1 * (double(zy) + sy));
                    vx = eh * (h3 * double(zx) + h * sx);
                    vy = eh * (h3 * double(zy) + h * sy);
                } else if (q == 3) {
                    zx = real(double(ax) + sx);
                    zy = real(double(ay) + sy);
                    vx = h6 * double(zx);
                    vy = h6 * double(zy);
                } else {
                    ax = real(double(ax) + eh * sx);
                    ay = real(double(ay) + eh * sy);
                    vx = q == 1 ? h3 * eh * double(zx) + h2 * sx : h6 * e1 * double(zx) + h2 * eh * sx;
                    vy = q == 1 ? h3 * eh * double(zy) + h2 * sy : h6 * e1 * double(zy) + h2 * eh * sy;
                }
                s.S[tid] = cmk<C>(real(vx), real(vy));
            }
        }
    if (act) {
        g.y[o] = zx;
        g.y[o + 1] = zy;
    }
}

// The first wavefront transforms both rows (row 0 + i row 1); wavefront f multiplies by
// base field f and transforms the products.
template <typename real, int N>
__device__ void flow_row_adj(const FlowArgs<real>& g, FlowLds<real, N>& s, int p) {
    using C = cplx<real>;
    using G = FlowGeo<real, N>;
    using T = LaneFft<real, N>;
    constexpr int M = G::M, MC = G::MC, KI = G::KI, R = T::R, L = T::L;
    const int tid = int(threadIdx.x), lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave), y0 = 2 * p;
    FlowWait wt{g.failed, g.polls};
    const FlowBuf rows = flow_buf(g.toRows, G::words(1)), cols = flow_buf(g.toCols, G::words(4));
    T ft;
    ft.init(g.tw);
    real b[R][2];
    flow_base(g, ft, wv, y0, b);
    unsigned src[2 * KI];
#pragma unroll
    for (int i = 0; i < 2 * KI; ++i) {
        const int k = lane + kWave * (i >> 1);
        src[i] = G::row_at(1, 0, y0 + (i & 1), k <= M ? k : M);
    }
    for (int t = MC + tid; t < N - M; t += 4 * kWave) s.A[0][t] = cmk<C>(real(0), real(0));
    __syncthreads();
    unsigned tag = g.tag;
    for (int n = 0; n < 4 * g.nsteps; ++n, ++tag) {
        C v[R];
        if (wv == 0) {
            flow_unpair<real, N, 1>(rows, src, tag, wt, s.A[0], lane);
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = s.A[0][ft.l + L * r];
            ft.template dif<+1>(v);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane < L) s.B[0][lane + L * r] = v[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const C z = s.B[0][ft.l + L * r];
            v[r] = cmk<C>(b[r][0] * z.x, b[r][1] * z.y);
        }
        ft.template dit<-1>(v);
        flow_split<real, N>(cols, ft, v, wv == 0 ? s.B[1] : s.A[wv], 4, wv, y0, tag, lane);
    }
}

template <typename real, int N> __global__ __launch_bounds__(4 * kWave, 4) void k_flow_adj(FlowArgs<real> g) {
    __shared__ FlowLds<real, N> s;
    const int b = int(blockIdx.x);
    if (b < FlowGeo<real, N>::MC)
        flow_col_adj<real, N>(g, s, b);
    else
        flow_row_adj<real, N>(g, s, b - FlowGeo<real, N>::MC);
}

}  // namespace tsk
