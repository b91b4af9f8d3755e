// Linear complex Ginzburg-Landau operator and its Crank-Nicolson time stepper.
//
// Equation (Sec. 2.3.2, eq. "ginzburg-landau equation"):
//     du/dt = -nu u_x + gamma u_xx + mu(x) u,  mu(x) = mu0 - c_u^2 + mu2 x^2 / 2,
// with nu = U + 2 i c_u and gamma = 1 + i c_d.  Second-order central
// differences on n interior nodes (Dirichlet ends) give the tridiagonal L_h;
// one matvec of M = exp(L T) is T/dt Crank-Nicolson steps
//     (I - dt/2 L_h) u+ = (I + dt/2 L_h) u.
//
// With A = I - dt/2 L_h the step is u+ = A^-1 (2 I - A) u = x - u, A x = 2 u: one
// tridiagonal solve and no explicit stencil.
//
// Two integrations:
//  * stepping (k_cgle_cn): the whole state (n <= 1024 complex128, 16 KB) stays in
//    one workgroup for the full integration, one thread per node.  The solve is
//    parallel cyclic reduction (Hockney & Jesshope): level l eliminates the
//    couplings at distance 2^l.  The elimination multipliers of the constant matrix
//    are computed once on the host when the parameters are set.  The matrix is
//    strictly diagonally dominant, so no pivoting is needed, and the multipliers
//    of level l fall like r^(2^l): the levels whose multipliers are all below 2^-64
//    change nothing and are left out (4 of 8 levels remain at 256 nodes on
//    [-50, 50], dt = 0.01).  A level costs an LDS write, a barrier and a read (about
//    330 cycles) and little arithmetic, so two levels are taken in one exchange: six
//    neighbours with the multiplied-out coefficients.  The increment u+ - u is
//    accumulated apart from u, so a step rounds the state once.  256 nodes: 1.27 us
//    a step with every level and the stencil, 0.55 with the levels that matter.
//  * squaring (cpower.hpp): the propagator of one step as a dense matrix, its
//    powers on the matrix cores of the whole device: log2(nsteps) launches
//    instead of nsteps dependent solves of one compute unit.
#include <algorithm>
#include <complex>
#include <vector>

#include "cpower.hpp"
#include "krylov.hpp"
#include "ops.hpp"

namespace tsk {

namespace {

constexpr int kCgleMaxN = 1024;
constexpr int kCgleMaxLevels = 10;

// One Crank-Nicolson integration (one workgroup).  Propagator: nsteps steps of
// the state in.  Forced (the resolvent mode): in is the forcing f^ of
// u' = L u + f^ e^{i omega t}; the run starts from rest, the forcing enters by
// the trapezoidal rule (dt/2 (f_n + f_{n+1}) = c1 e^{i omega t_n} f^ with
// c1 = dt/2 (1 + e^{i omega dt})), and the output is the phase-normalised state
// u(t_N) e^{-i omega t_N}.
struct CnJob {
    const double2* in;    // input of Krylov step j: in + j * in_stride
    long long in_stride;  // elements (0: one fixed input)
    double2* out;
    // alpha[levels n] | gamma[levels n] | binv[n] | binv - 1 [n] | dt/2 main[n] | pairs[6 (levels/2) n]
    const double2* tab;
    const double2* tabh;  // the tables of the conjugate transpose
    double2 sub, sup;     // dt/2 times the constant sub/super diagonals of L_h
    double2 c1;
    double omega, dt;
    int n, levels, levelsh, nsteps, forced;
};

__device__ __forceinline__ double lane_bcast(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(int(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane(int(b >> 32), lane);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
    return cmk<double2>(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}

// LV = the number of reduction levels (the largest of a batch): a compile-time count
// keeps the multipliers in registers.  NB neighbours per side of an exchange: 3
// (two levels each; the last of an odd count alone), or 1 with more than 512
// threads, whose reads of three would keep the LDS busy longer than a second
// exchange takes (1000 nodes, 6 levels: 1.60 us a step with 3, 1.28 with 1).
template <int LV, int NT>
__device__ __forceinline__ void cn_integrate(const CnJob& jb, int j) {
    __shared__ double2 bufA[NT];
    __shared__ double2 bufB[NT];
    constexpr int NB = NT > 512 ? 1 : 3;
    constexpr int NX = NB == 3 ? (LV + 1) / 2 : LV;  // exchanges per step
    const int n = jb.n;
    const int i = threadIdx.x;
    const bool act = i < n;
    const double2 zero = cmk<double2>(0.0, 0.0);
    const double2* __restrict__ alpha = jb.tab;
    const double2* __restrict__ gamma = alpha + size_t(jb.levels) * n;
    const double2* __restrict__ binv = gamma + size_t(jb.levels) * n;
    const double2* __restrict__ pairs = binv + size_t(3) * n;
    // coefficients of the neighbours i -+ s (c + 1); an integration of fewer levels
    // than LV has zeros beyond them, which change nothing.  Out-of-range neighbours
    // have zero coefficients too: the index is clamped instead of branching (the
    // state is finite, so 0 * x = 0 exactly).
    double2 lo[NX][NB], hi[NX][NB];
    int im[NX][NB], ip[NX][NB];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const int l = NB == 3 ? 2 * x : x;  // first level of the exchange
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            im[x][c] = max(i - (c + 1) * (1 << l), 0);
            ip[x][c] = min(i + (c + 1) * (1 << l), n - 1);
            lo[x][c] = hi[x][c] = zero;
            if (act && NB == 3 && l + 1 < jb.levels) {
                lo[x][c] = pairs[size_t(6 * x + c) * n + i];
                hi[x][c] = pairs[size_t(6 * x + 3 + c) * n + i];
            } else if (act && c == 0 && l < jb.levels) {
                lo[x][c] = alpha[size_t(l) * n + i];
                hi[x][c] = gamma[size_t(l) * n + i];
            }
        }
    }
    const double2 bi = act ? binv[i] : zero, bm = act ? binv[n + i] : zero;
    const double2* __restrict__ uin = jb.in + j * jb.in_stride;
    const bool forced = jb.forced != 0;
    const double2 fh = (forced && act) ? cscale(cmul(jb.c1, uin[i]), 0.5) : zero;
    double2 u = (!forced && act) ? uin[i] : zero;
    // forcing phases e^{i omega dt s}: lane l of every wave evaluates step s0 + l
    // once per 64 steps, step s reads lane s - s0
    const int lane = i & (kWave - 1);
    double2 ph = zero;
    double2* src = bufA;
    double2* dst = bufB;
    for (int st = 0; st < jb.nsteps; ++st) {
        // x = A^-1 (u + f/2), f the step's forcing; the right-hand side is u + t
        double2 t = zero;
        if (forced) {
            if ((st & (kWave - 1)) == 0) {
                double sn, cs;
                sincos(jb.omega * jb.dt * double(st + lane), &sn, &cs);
                ph = cmk<double2>(cs, sn);
            }
            const int sl = st & (kWave - 1);  // uniform, < 64
            const double2 e = cmk<double2>(lane_bcast(ph.x, sl), lane_bcast(ph.y, sl));
            t = cmul(e, fh);
        }
        // two LDS buffers in turn: a buffer is written again only after the barrier
        // that every reader of its last contents has passed
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            double2* sw = src;
            src = dst;
            dst = sw;
            src[i] = cadd(u, t);
            __syncthreads();
            double2 vl[NB], vh[NB];
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                vl[c] = src[im[x][c]];
                vh[c] = src[ip[x][c]];
            }
            // (the last exchange of an odd level count has one neighbour per side)
            const int used = NB == 3 && 2 * x + 1 >= LV ? 1 : NB;
            double2 a = cmul(lo[x][0], vl[0]), b = cmul(hi[x][0], vh[0]);
#pragma unroll
            for (int c = 1; c < NB; ++c)
                if (c < used) {
                    a = cfma(lo[x][c], vl[c], a);
                    b = cfma(hi[x][c], vh[c], b);
                }
            t = cadd(t, cadd(a, b));
        }
        // u+ = 2 x - u = u + 2 (t binv + u (binv - 1))
        const double2 d = cfma(t, bi, cmul(u, bm));
        u = cmk<double2>(fma(2.0, d.x, u.x), fma(2.0, d.y, u.y));
    }
    if (forced) {
        double sn, cs;
        sincos(jb.omega * jb.dt * double(jb.nsteps), &sn, &cs);
        u = cmul(u, cmk<double2>(cs, -sn));
    }
    if (act) jb.out[i] = u;
}

template <int LV, int NT>
__global__ __launch_bounds__(NT) void k_cgle_cn(CnJob jb) { cn_integrate<LV, NT>(jb, 0); }

// A batch of integrations (one per workgroup), Krylov step j of each.
template <int LV, int NT>
__global__ __launch_bounds__(NT) void k_cgle_cn_batch(const CnJob* __restrict__ jobs, int j) {
    const CnJob jb = jobs[blockIdx.x];
    cn_integrate<LV, NT>(jb, j);
}

// Launch with the level count as a template argument (jobs == null: the single
// job `one`).
template <int LV, int NT>
void launch_cn_nt(const CnJob& one, const CnJob* jobs, int count, int j, int threads, hipStream_t s) {
    if (jobs)
        hipLaunchKernelGGL((k_cgle_cn_batch<LV, NT>), dim3(count), dim3(threads), 0, s, jobs, j);
    else
        hipLaunchKernelGGL((k_cgle_cn<LV, NT>), dim3(1), dim3(threads), 0, s, one);
}
template <int LV>
void launch_cn(const CnJob& one, const CnJob* jobs, int count, int j, int threads, hipStream_t s) {
    if (threads <= 512)
        launch_cn_nt<LV, 512>(one, jobs, count, j, threads, s);
    else
        launch_cn_nt<LV, kCgleMaxN>(one, jobs, count, j, threads, s);
}

tsk_status launch_cn_levels(int levels, const CnJob& one, const CnJob* jobs, int count, int j, int threads,
                            hipStream_t s) {
    if (levels < 1 || levels > kCgleMaxLevels || threads > kCgleMaxN || threads % kWave)
        return fail(TSK_EINVAL, "CGLE launch shape does not fit the reduction depth");
    switch (levels) {
        case 1: launch_cn<1>(one, jobs, count, j, threads, s); break;
        case 2: launch_cn<2>(one, jobs, count, j, threads, s); break;
        case 3: launch_cn<3>(one, jobs, count, j, threads, s); break;
        case 4: launch_cn<4>(one, jobs, count, j, threads, s); break;
        case 5: launch_cn<5>(one, jobs, count, j, threads, s); break;
        case 6: launch_cn<6>(one, jobs, count, j, threads, s); break;
        case 7: launch_cn<7>(one, jobs, count, j, threads, s); break;
        case 8: launch_cn<8>(one, jobs, count, j, threads, s); break;
        case 9: launch_cn<9>(one, jobs, count, j, threads, s); break;
        case 10: launch_cn<10>(one, jobs, count, j, threads, s); break;
        default: return fail(TSK_EINVAL, "CGLE reduction depth out of range");
    }
    TSK_HIP(hipGetLastError());
    return TSK_OK;
}

// ---- the one-step matrix for squaring ------------------------------------------------------
// D = e S - I with S = A^-1 (2 I - A) and e = e^{-i omega dt} (resolvent mode: the
// step of v = u e^{-i omega t}; else e = 1): S - I = A^-1 dt L_h commutes with L_h,
// so row i of it is the conjugate of A^-H (dt L_h^H)[:, i], one solve with the
// transposed tables whose result is contiguous in memory.  D = e (S - I) + (e - 1) I
// keeps the small matrix to full relative accuracy.  A workgroup solves R rows at
// once, sharing the loads of the multipliers; rows and columns from n to ld are
// zeroed; b = 1 (cpower.hpp).  The workgroup after the last rows sets the vectors:
// propagator v = x, q = 0; resolvent v = 0, q = e A^-1 c1 f.
struct CpowForm {
    double* D;    // [count][cpow_stride]
    double* vec;  // [count][4][ld]
    int ld;
};
template <int R>
__global__ __launch_bounds__(kCgleMaxN) void k_cgle_form(CnJob one, const CnJob* __restrict__ jobs, int jstep,
                                                         CpowForm f) {
    extern __shared__ double2 lds_form[];  // [2][R][threads]
    const int nt = int(blockDim.x), t = int(threadIdx.x), ld = f.ld, m = int(blockIdx.y);
    const CnJob jb = jobs ? jobs[m] : one;
    const int n = jb.n, rowblocks = (ld + R - 1) / R;
    const bool vecs = int(blockIdx.x) == rowblocks;
    const double2 zero = cmk<double2>(0.0, 0.0);
    const bool act = t < n;
    const bool forced = jb.forced != 0;
    // e and e - 1
    double2 e = cmk<double2>(1.0, 0.0), em = zero;
    if (forced) {
        double sn, cs, s2, c2;
        sincos(jb.omega * jb.dt, &sn, &cs);
        sincos(0.5 * jb.omega * jb.dt, &s2, &c2);
        e = cmk<double2>(cs, -sn);
        em = cmk<double2>(-2.0 * s2 * s2, -sn);
    }
    double* vec = f.vec + size_t(4 * ld) * m;
    const double2* in = jb.in + jstep * jb.in_stride;
    if (vecs && !forced) {
        if (t < ld) {
            const double2 u = act ? in[t] : zero;
            vec[t] = u.x;
            vec[ld + t] = u.y;
            vec[2 * ld + t] = vec[3 * ld + t] = 0.0;
        }
        return;
    }
    const int levels = vecs ? jb.levels : jb.levelsh;
    const double2* __restrict__ al = vecs ? jb.tab : jb.tabh;
    const double2* __restrict__ ga = al + size_t(levels) * n;
    const double2* __restrict__ bi = ga + size_t(levels) * n;
    const double2* __restrict__ hm = jb.tab + size_t(2 * jb.levels + 2) * n;  // dt/2 main of L_h
    double2 d[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        d[r] = zero;
        const int i = int(blockIdx.x) * R + r;
        if (vecs) {
            if (r == 0 && act) d[0] = cmul(jb.c1, in[t]);
        } else if (i < n && act) {  // dt (L_h^H)[t][i] = dt conj(L_h[i][t])
            const double2 a = t == i ? hm[i] : t == i - 1 ? jb.sub : t == i + 1 ? jb.sup : zero;
            d[r] = cmk<double2>(2.0 * a.x, -2.0 * a.y);
        }
    }
    double2* src = lds_form;
    double2* dst = lds_form + R * nt;
    for (int l = 0; l < levels; ++l) {
        double2* sw = src;
        src = dst;
        dst = sw;
#pragma unroll
        for (int r = 0; r < R; ++r) src[r * nt + t] = d[r];
        __syncthreads();
        if (act) {
            const double2 a = al[size_t(l) * n + t], g = ga[size_t(l) * n + t];
            const int tm = max(t - (1 << l), 0), tp = min(t + (1 << l), n - 1);
#pragma unroll
            for (int r = 0; r < R; ++r)
                d[r] = cadd(d[r], cadd(cmul(a, src[r * nt + tm]), cmul(g, src[r * nt + tp])));
        }
    }
    if (t >= ld) return;
    const double2 b = act ? bi[t] : zero;
    if (vecs) {
        const double2 q = cmul(e, cmul(b, d[0]));
        vec[t] = vec[ld + t] = 0.0;
        vec[2 * ld + t] = q.x;
        vec[3 * ld + t] = q.y;
        return;
    }
    double* Dm = f.D + cpow_stride(ld) * m;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = int(blockIdx.x) * R + r;
        if (i >= ld) continue;
        double2 x = zero;
        if (i < n && act) {
            x = cmul(e, cconj(cmul(b, d[r])));
            if (t == i) x = cadd(x, em);
        }
        if (t == i) Dm[2 * size_t(ld) * ld + i] = 1.0;
        Dm[size_t(i) * ld + t] = x.x;
        Dm[size_t(ld) * ld + size_t(i) * ld + t] = x.y;
    }
}

// Stepping or squaring, from estimated times in us: a step is one exchange after the
// other (256 nodes, 4 levels 0.39, 400 nodes 0.51, 1000 nodes, 6 levels 1.28), forming the
// matrix 8, doublings and applications as in cpower.hpp.  100 steps at 256 nodes: 41
// stepping, 106 squaring; 23000 steps at 400 nodes: 13100 and 340.  The rule looks at one
// integration alone, so a batch gives the bits of single runs.
struct CnPlan {
    bool square = false;
    int doublings = 0;
};
inline CnPlan cn_plan(const CnJob& jb) {
    const double n = jb.n;
    const double step = jb.n <= 512 ? ((jb.levels + 1) / 2) * (0.13 + 0.0003 * n) : 0.2 * jb.levels;
    const CpowCost c{CpowWork::ld_of(jb.n, 1), 1, CpowWork::tiles_of(jb.n, 1), false};
    double cost = 0.0;
    CnPlan p;
    p.doublings = c.doublings(jb.nsteps, c.ld, &cost);
    p.square = 8.0 + cost < 0.8 * step * jb.nsteps;
    return p;
}

// Tables of one Crank-Nicolson propagator: the cyclic-reduction multipliers of the
// implicit matrix, level by level and multiplied out for pairs of levels, and dt/2
// times the diagonals of L_h.
struct CnTables {
    double2 sub{}, sup{};
    int levels = 0;
    DevBuf tab;  // as CnJob::tab
};

// count integrations of one node and step count by squaring (jobs: device table, or
// the single job `one`).
tsk_status cn_square(const CpowWork& W, const CnPlan& p, const CnJob& one, const CnJob* jobs, int count, int j,
                     int threads, bool forced, const CpowOut<double>& out, hipStream_t s) {
    const CpowForm f{W.D<double>(0), W.v<double>(0), W.ld};
    const int nt = std::max(threads, (W.ld + kWave - 1) / kWave * kWave);
    if (nt <= 512)
        hipLaunchKernelGGL(k_cgle_form<4>, dim3((W.ld + 3) / 4 + 1, count), dim3(nt), 2 * 4 * nt * sizeof(double2), s,
                           one, jobs, j, f);
    else
        hipLaunchKernelGGL(k_cgle_form<2>, dim3((W.ld + 1) / 2 + 1, count), dim3(nt), 2 * 2 * nt * sizeof(double2), s,
                           one, jobs, j, f);
    return cpow_run<double>(W, one.nsteps, forced, W.ld, p.doublings, out, s);
}

struct CgleOp final : Operator {
    int nn = 0;
    double half_width = 0.0;
    int nsteps = 0;
    double dt = 0.0;
    CnTables fwd, adj;  // L_h and its conjugate transpose (the adjoint propagator)
    // resolvent mode: apply = R(omega) by ntrans forced steps from rest
    bool resolvent = false;
    double omega = 0.0, ttrans = 0.0;
    int ntrans = 0;

    const char* name() const override { return "cgle1d"; }
    int64_t physical_reals() const override { return 2 * int64_t(nn); }

    tsk_status set_params(double U, double c_u, double c_d, double mu0, double mu2, double dt, double TT) {
        using cd = std::complex<double>;
        if (!(dt > 0.0) || !(TT > 0.0) || !std::isfinite(dt) || !std::isfinite(TT))
            return fail(TSK_EINVAL, "dt and T must be positive and finite");
        double ns = TT / dt;
        int nsi = int(std::lround(ns));
        if (nsi < 1 || std::fabs(ns - nsi) > 1e-9 * std::max(1.0, ns))
            return fail(TSK_EINVAL, "T must be an integer multiple of dt");
        const int n_ = nn;
        const double dx = 2.0 * half_width / (n_ + 1);
        const cd nu(U, 2.0 * c_u), gam(1.0, c_d);
        const cd sub = gam / (dx * dx) + nu / (2.0 * dx);
        const cd sup = gam / (dx * dx) - nu / (2.0 * dx);
        std::vector<cd> mainv(n_), mainh(n_);
        for (int j = 0; j < n_; ++j) {
            double x = -half_width + dx * (j + 1);
            double mux = (mu0 - c_u * c_u) + mu2 * x * x / 2.0;
            mainv[j] = -2.0 * gam / (dx * dx) + mux;
            mainh[j] = std::conj(mainv[j]);
        }
        int L = 0;
        while ((1 << L) < n_) ++L;
        // L_h^H: conjugated main diagonal, sub and super diagonals swapped and conjugated
        TSK_TRY(build(fwd, sub, sup, mainv, 0.5 * dt, L));
        TSK_TRY(build(adj, std::conj(sup), std::conj(sub), mainh, 0.5 * dt, L));
        nsteps = nsi;
        T = TT;
        this->dt = dt;
        if (resolvent) ntrans = std::max(1, int(std::lround(ttrans / dt)));
        params_set = true;
        return TSK_OK;
    }

    // Crank-Nicolson tables of the tridiagonal (sub, mainv, sup), h = dt/2.
    tsk_status build(CnTables& tb, std::complex<double> sub, std::complex<double> sup,
                     const std::vector<std::complex<double>>& mainv, double h, int L) {
        using cd = std::complex<double>;
        const int n_ = nn;
        std::vector<cd> a(n_), b(n_), c(n_), bd(n_);
        for (int j = 0; j < n_; ++j) {
            a[j] = j > 0 ? -h * sub : cd(0.0);
            bd[j] = -h * mainv[j];  // b - 1, kept apart: it is small
            b[j] = 1.0 + bd[j];
            c[j] = j + 1 < n_ ? -h * sup : cd(0.0);
        }
        // levels until every multiplier is below 2^-64: a level left out would change
        // the solution by less than 2^-63 of its largest value
        const double tiny = 0x1.0p-64;
        std::vector<cd> al, ga;
        int lv = 0;
        for (int l = 0, s = 1; l < L; ++l, s <<= 1) {
            std::vector<cd> a2(n_), b2(n_), c2(n_), bd2(n_), av(n_), gv(n_);
            double big = 0.0;
            for (int j = 0; j < n_; ++j) {
                cd alpha = j - s >= 0 ? -a[j] / b[j - s] : cd(0.0);
                cd gamma = j + s < n_ ? -c[j] / b[j + s] : cd(0.0);
                av[j] = alpha;
                gv[j] = gamma;
                const double m = std::max(std::abs(alpha), std::abs(gamma));
                if (!(m <= big)) big = m;  // NaN counts as big
                a2[j] = j - s >= 0 ? alpha * a[j - s] : cd(0.0);
                c2[j] = j + s < n_ ? gamma * c[j + s] : cd(0.0);
                bd2[j] = bd[j] + (j - s >= 0 ? alpha * c[j - s] : cd(0.0)) + (j + s < n_ ? gamma * a[j + s] : cd(0.0));
                b2[j] = 1.0 + bd2[j];
            }
            if (l > 0 && big < tiny) break;
            al.insert(al.end(), av.begin(), av.end());
            ga.insert(ga.end(), gv.begin(), gv.end());
            ++lv;
            a.swap(a2); b.swap(b2); c.swap(c2); bd.swap(bd2);
        }
        std::vector<double2> host;
        host.reserve(size_t(n_) * (3 + 5 * size_t(lv)));
        auto put = [&](cd v) { host.push_back(cmk<double2>(v.real(), v.imag())); };
        for (const cd& v : al) put(v);
        for (const cd& v : ga) put(v);
        for (int j = 0; j < n_; ++j) put(1.0 / b[j]);
        for (int j = 0; j < n_; ++j) put(-bd[j] / b[j]);
        for (int j = 0; j < n_; ++j) put(h * mainv[j]);
        // levels l, l + 1 in one exchange: with d'_j = d_j + al_j d_{j-s} + ga_j d_{j+s} the second
        // level's d'_i + al2_i d'_{i-2s} + ga2_i d'_{i+2s} in terms of d at i +- s, 2s, 3s
        for (int l = 0; l + 1 < lv; l += 2) {
            const int s = 1 << l;
            auto at = [&](const std::vector<cd>& v, int lev, int j) {
                return j >= 0 && j < n_ ? v[size_t(lev) * n_ + j] : cd(0.0);
            };
            for (int c = 0; c < 6; ++c)
                for (int j = 0; j < n_; ++j) {
                    const cd a2 = at(al, l + 1, j), g2 = at(ga, l + 1, j);
                    if (c == 0) put(at(al, l, j) + a2 * at(ga, l, j - 2 * s));
                    else if (c == 1) put(a2);
                    else if (c == 2) put(a2 * at(al, l, j - 2 * s));
                    else if (c == 3) put(at(ga, l, j) + g2 * at(al, l, j + 2 * s));
                    else if (c == 4) put(g2);
                    else put(g2 * at(ga, l, j + 2 * s));
                }
        }
        TSK_TRY(tb.tab.ensure(host.size() * sizeof(double2)));
        TSK_HIP(hipMemcpy(tb.tab.ptr, host.data(), host.size() * sizeof(double2), hipMemcpyHostToDevice));
        cd rs = h * sub, rp = h * sup;
        tb.sub = cmk<double2>(rs.real(), rs.imag());
        tb.sup = cmk<double2>(rp.real(), rp.imag());
        tb.levels = lv;
        return TSK_OK;
    }

    // Propagator (forced = false: T/dt steps of x) or resolvent (forced = true:
    // x is the forcing, ntrans steps at frequency w from rest).
    CnJob job(bool adjoint, bool forced, double w) const {
        const CnTables &tb = adjoint ? adj : fwd, &th = adjoint ? fwd : adj;
        CnJob jb{};
        jb.tab = tb.tab.as<double2>();
        jb.tabh = th.tab.as<double2>();
        jb.sub = tb.sub;
        jb.sup = tb.sup;
        jb.n = nn;
        jb.levels = tb.levels;
        jb.levelsh = th.levels;
        jb.dt = dt;
        jb.forced = forced ? 1 : 0;
        if (forced) {
            const double h = 0.5 * dt;
            jb.c1 = cmk<double2>(h * (1.0 + std::cos(w * dt)), h * std::sin(w * dt));
            jb.omega = w;
            jb.nsteps = ntrans;
        } else {
            jb.nsteps = nsteps;
        }
        return jb;
    }
    int threads() const { return (nn + kWave - 1) / kWave * kWave; }
    tsk_status run(bool adjoint, const void* x, void* y) {
        if (!ready()) return fail(TSK_ESTATE, "CGLE parameters not set");
        if (x == y) return fail(TSK_EINVAL, "input and output must not alias");
        CnJob jb = job(adjoint, resolvent, adjoint ? -omega : omega);
        jb.in = static_cast<const double2*>(x);
        jb.out = static_cast<double2*>(y);
        const CnPlan p = cn_plan(jb);
        CpowWork W;
        if (p.square && W.place(scratch(), stream, nn, 1, sizeof(double), 2, 0)) {
            CpowOut<double> out{reinterpret_cast<double*>(y), 0, nullptr, nn};
            return cn_square(W, p, jb, nullptr, 1, 0, threads(), resolvent, out, stream);
        }
        return launch_cn_levels(jb.levels, jb, nullptr, 1, 0, threads(), stream);
    }
    tsk_status apply(const void* x, void* y) override { return run(false, x, y); }
    // M^H: Crank-Nicolson with L_h^H (the two factors of a step commute, so this is
    // the conjugate transpose of the forward propagator).  Resolvent mode:
    // R(omega)^H = the forced integration with L_h^H at frequency -omega.
    tsk_status apply_adjoint(const void* x, void* y) override { return run(true, x, y); }
    bool has_adjoint() const override { return true; }
    tsk_status from_physical(const void* phys, void* state) override {
        TSK_HIP(hipMemcpyAsync(state, phys, state_bytes(), hipMemcpyDeviceToDevice, stream));
        return TSK_OK;
    }
    tsk_status to_physical(const void* state, void* phys) override {
        TSK_HIP(hipMemcpyAsync(phys, state, state_bytes(), hipMemcpyDeviceToDevice, stream));
        return TSK_OK;
    }
};

}  // namespace

tsk_status make_cgle(int n, double half_width, hipStream_t s, std::unique_ptr<Operator>* out) {
    if (n < 2 || n > kCgleMaxN) return fail(TSK_EINVAL, "CGLE node count must be in [2, 1024]");
    if (!(half_width > 0.0) || !std::isfinite(half_width)) return fail(TSK_EINVAL, "half_width must be positive");
    auto op = std::make_unique<CgleOp>();
    op->nn = n;
    op->half_width = half_width;
    op->n = n;
    op->kind = StateKind::Complex64x2;
    op->stream = s;
    op->base_set = true;  // the CGLE has no base flow
    *out = std::move(op);
    return TSK_OK;
}

tsk_status cgle_set_params(Operator* op, double U, double c_u, double c_d, double mu0, double mu2, double dt,
                           double T) {
    auto* c = dynamic_cast<CgleOp*>(op);
    if (!c) return fail(TSK_EINVAL, "not a Ginzburg-Landau operator");
    return c->set_params(U, c_u, c_d, mu0, mu2, dt, T);
}

bool is_cgle(const Operator* op) { return dynamic_cast<const CgleOp*>(op) != nullptr; }

tsk_status cgle_set_resolvent(Operator* op, double omega, double t_transient) {
    auto* c = dynamic_cast<CgleOp*>(op);
    if (!c) return fail(TSK_EINVAL, "the resolvent mode needs a Ginzburg-Landau operator (complex state)");
    if (!c->params_set) return fail(TSK_ESTATE, "CGLE parameters not set");
    if (!std::isfinite(omega) || !std::isfinite(t_transient) || t_transient < 0.0)
        return fail(TSK_EINVAL, "omega must be finite and t_transient >= 0");
    if (t_transient == 0.0) {
        c->resolvent = false;
        return TSK_OK;
    }
    const double steps = t_transient / c->dt;
    if (!(steps >= 0.5) || steps > 1e9)
        return fail(TSK_EINVAL, "t_transient must span between one and 1e9 time steps");
    c->resolvent = true;
    c->omega = omega;
    c->ttrans = t_transient;
    c->ntrans = int(std::lround(steps));
    return TSK_OK;
}

// ---- batches: all instances of a pass in one stepping launch (one workgroup per
// instance) or, by the rule of a single integration, squared together where node
// and step count agree ---------------------------------------------------------------
struct CgleBatch {
    struct Square {
        CnPlan plan;
        CnJob first;
        DevBuf jobs, outs;  // job table and output addresses of the group
        int count = 0;
    };
    struct Pass {
        DevBuf jobs;  // the stepping instances
        int count = 0, levels = 1;
        std::vector<std::unique_ptr<Square>> squares;
    };
    Pass first, second;  // V -> out (or tmp), and (M^H M) tmp -> w
    Operator* lead = nullptr;  // squares in its scratch; null: step
    int n = 0, chunk = 1, threads = 0;
    bool two = false;
};

void cgle_batch_free(CgleBatch* b) { delete b; }

namespace {

tsk_status cgle_pass_plan(CgleBatch* b, const std::vector<CnJob>& jobs, CgleBatch::Pass* p) {
    std::vector<CnJob> step;
    std::vector<std::vector<CnJob>> sq;
    for (const CnJob& jb : jobs) {
        if (!b->lead || !cn_plan(jb).square) {
            step.push_back(jb);
            p->levels = std::max(p->levels, jb.levels);
            continue;
        }
        size_t q = 0;
        while (q < sq.size() && (sq[q][0].nsteps != jb.nsteps || sq[q][0].forced != jb.forced)) ++q;
        if (q == sq.size()) sq.push_back({});
        sq[q].push_back(jb);
    }
    p->count = int(step.size());
    if (p->count > 0) {
        TSK_TRY(p->jobs.ensure(sizeof(CnJob) * step.size()));
        TSK_HIP(hipMemcpy(p->jobs.ptr, step.data(), sizeof(CnJob) * step.size(), hipMemcpyHostToDevice));
    }
    for (const auto& g : sq) {
        auto s = std::make_unique<CgleBatch::Square>();
        std::vector<double2*> outs;
        for (const CnJob& jb : g) outs.push_back(jb.out);
        s->plan = cn_plan(g[0]);
        s->first = g[0];
        s->count = int(g.size());
        TSK_TRY(s->jobs.ensure(sizeof(CnJob) * g.size()));
        TSK_HIP(hipMemcpy(s->jobs.ptr, g.data(), sizeof(CnJob) * g.size(), hipMemcpyHostToDevice));
        TSK_TRY(s->outs.ensure(sizeof(double2*) * g.size()));
        TSK_HIP(hipMemcpy(s->outs.ptr, outs.data(), sizeof(double2*) * g.size(), hipMemcpyHostToDevice));
        p->squares.push_back(std::move(s));
    }
    return TSK_OK;
}

tsk_status cgle_pass_run(CgleBatch* b, const CgleBatch::Pass& p, int j, hipStream_t s) {
    if (p.count > 0)
        TSK_TRY(launch_cn_levels(p.levels, CnJob{}, p.jobs.as<CnJob>(), p.count, j, b->threads, s));
    for (const auto& g : p.squares)
        for (int c = 0; c < g->count; c += b->chunk) {
            const int cnt = std::min(b->chunk, g->count - c);
            CpowWork W;
            if (!W.place(b->lead->scratch(), s, b->n, cnt, sizeof(double), 2, 0))
                return fail(TSK_ENOMEM, "no memory for a squared Ginzburg-Landau batch");
            const CpowOut<double> out{nullptr, 0, g->outs.as<double*>() + c, b->n};
            TSK_TRY(cn_square(W, g->plan, g->first, g->jobs.as<CnJob>() + c, cnt, j, b->threads,
                              g->first.forced != 0, out, s));
        }
    return TSK_OK;
}

}  // namespace

tsk_status cgle_batch_plan(Operator* const* ops, int count, const KryDesc* D_host, bool svd, CgleBatchPtr* out) {
    out->reset();
    std::vector<CnJob> a(count), b(count);
    auto* c0 = dynamic_cast<CgleOp*>(ops[0]);
    if (!c0) return fail(TSK_EINVAL, "not a Ginzburg-Landau batch");
    for (int i = 0; i < count; ++i) {
        const auto* c = dynamic_cast<const CgleOp*>(ops[i]);
        if (!c || !c->ready()) return fail(TSK_ESTATE, "batch member is not a ready Ginzburg-Landau operator");
        if (c->nn != c0->nn) return TSK_OK;  // mixed sizes: per-instance launches
        const KryDesc& d = D_host[i];
        void* mid = svd ? ops[i]->aw.tmp.ptr : d.w;
        if (!d.V || !mid || !d.w) return fail(TSK_EINVAL, "batch workspace not allocated");
        a[i] = c->job(false, c->resolvent, c->omega);
        a[i].in = static_cast<const double2*>(d.V);
        a[i].in_stride = d.ldv;
        a[i].out = static_cast<double2*>(mid);
        if (svd) {
            b[i] = c->job(true, c->resolvent, -c->omega);
            b[i].in = static_cast<const double2*>(mid);
            b[i].in_stride = 0;
            b[i].out = static_cast<double2*>(d.w);
        }
    }
    auto p = CgleBatchPtr(new CgleBatch);
    p->n = c0->nn;
    p->threads = c0->threads();
    p->two = svd;
    // matrices squared at once: at most 1 GiB of them
    const size_t each = 2 * CpowWork::bytes((c0->nn + 31) / 32 * 32, sizeof(double));
    p->chunk = int(std::min<size_t>(size_t(count), std::max<size_t>(1, (size_t(1) << 30) / each)));
    bool any = false;
    for (int i = 0; i < count; ++i) any = any || cn_plan(a[i]).square || (svd && cn_plan(b[i]).square);
    // (smaller groups have room in what the largest chunk has)
    CpowWork W;
    if (any && W.place(c0->scratch(), c0->stream, c0->nn, p->chunk, sizeof(double), 2, 0)) p->lead = c0;
    TSK_TRY(cgle_pass_plan(p.get(), a, &p->first));
    if (svd) TSK_TRY(cgle_pass_plan(p.get(), b, &p->second));
    *out = std::move(p);
    return TSK_OK;
}

tsk_status cgle_batch_matvec(CgleBatch* b, int j, hipStream_t s) {
    TSK_TRY(cgle_pass_run(b, b->first, j, s));
    if (b->two) TSK_TRY(cgle_pass_run(b, b->second, 0, s));
    return TSK_OK;
}

}  // namespace tsk
