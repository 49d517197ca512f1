// HIP kernels (gfx950) of the LAMP iteration: Algorithm 2 with the log-domain
// marginals of Section 4.1, for the cost C_ij = s ||x_i - y_j||^2 generated on
// the fly.
//
// Notation (all logarithms of probabilities are kept in base 2; LOG2E = 1/ln 2):
//   points are centred, x~_i = x_i - mu, y~_j = y_j - mu (C is translation
//   invariant), stored as FP64, with squared norms xn2_i, yn2_j;
//   for a dual vector v and inverse temperature lam (= 1/eta),
//     e_ij = -lam LOG2E (C_ij + K v_j)                                  K = 2||C||_inf
//          = q_i + g_j + cfac * (x~_i . y~_j)
//     q_i  = -lam LOG2E s xn2_i,  g_j = -lam LOG2E (s yn2_j + K v_j),  cfac = 2 s lam LOG2E.
//   The row log-normaliser (Section 4.1, first display) in base 2 is
//     l_i = q_i + sigma_i,   sigma_i = log2 sum_j 2^(g_j + cfac x~_i.y~_j).
//   Iteration t evaluates two couplings: A = p^{eta_t}(nu^t) and B = p^{eta_{t+1}}(nubar^{t+1}).
//
// Row sweep: a per-row offset h_i (in dot-product units) is shared by A and B;
//     S_i = sum_j 2^(cfac (h_i + x~_i.y~_j) + g_j) = 2^(cfac h_i + sigma_i).
// h_i is the previous iteration's -sigma^B_i / cfac^B, which keeps every
// exponent within a few units of 0 (the per-iteration change of the exponents
// is bounded by tau1 ||C||_inf-scaled terms); rows whose sums leave a safe range
// are recomputed exactly.  No running max is needed.
//
// Column sweep (Section 4.1, second display): with k_i = -sigma^B_i / cfac^B,
//     p^B_ij = 2^(cfac^B (k_i + x~.y~) + g^B_j)
//     p^A_ij = 2^(rho sigma^B_i - sigma^A_i) * 2^(cfac^A (k_i + x~.y~) + g^A_j),  rho = cfac^A/cfac^B,
// so col_j = sum_i w_i 2^(...) with per-row weights w^B_i = r_i, w^A_i = r_i 2^(rho sigma^B - sigma^A).
//
// Every (i, j) exponent is assembled in FP64 (full-rate FMA on CDNA4), converted
// to FP32 and exponentiated with v_exp_f32; sums run in FP32 within short chunks
// and are carried in FP64.  The streamed side of each sweep (columns for the row
// sweep, rows for the column sweep) is wave-uniform and is read through scalar
// loads; the owned side lives in VGPRs, one row (or column) per lane.  Partial
// sums over splits of the streamed range go to a workspace and are merged in a
// fixed order, so results are deterministic.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lampk {

constexpr double LOG2E = 1.4426950408889634074;
constexpr double LN2 = 0.69314718055994530942;
constexpr int BLOCK = 256;
constexpr int UNROLL = 8;

// Device-side control block (lives in the workspace).
struct Ctrl {
    int64_t t;          // index of the iteration the next kernels execute
    int64_t t_row;      // the same for the row sweep and row finish: ahead of t by one between the
                        // dual update of iteration t and its completion (complete_iteration)
    int64_t t_end;      // exclusive end of this call's iterations
    int64_t t_base;     // schedule index base: sched[t - t_base]
    int64_t t_done;     // iteration whose residual met tol (-1 otherwise)
    int32_t done;       // 1 once res_t <= tol
    int32_t err;        // bit 0: non-finite value in the dual update
    int32_t fallbacks;  // rows recomputed exactly, in the iterations whose dual update ran
    int32_t fallbacks_row;   // those of the running iteration
    int32_t done_seen;  // done as of the last dual update
    uint32_t pad0;
    double tol;         // 0: never stop early
    double res_last;    // ||col(X^t) - c||_1 of the last completed iteration
    double dt_acc;      // accumulated D_t summands without the normaliser telescope
    double dt_cost;     // <C, Xbar^{t+1}> of the running iteration (D_t tracking)
};

// Per-iteration scalars, filled on the host in FP64 by the recursion of step:eta_update.
struct Sched {
    double lamA;   // lam_t
    double lamB;   // lam_{t+1}
    double w;      // tau1 / lam_{t+1}  (= tau1 eta_{t+1})
    double lamC;   // lam_{t+2}
    double w2;     // tau1 / lam_{t+2}
    double pad[3];
};

// Per-solve constants.
struct Consts {
    int64_t n, m;
    double s;       // cost scale
    double K;       // 2 ||C||_inf
    double kappa;   // 2 tau2 ||C||_inf
    double alpha_m; // alpha / m
    double clipb;   // tanh(beta / 2)
    int metric;     // ground cost, METRIC_*
    int factor_cols;     // one-chain matrix-core column sweep: per-column factor (see there)
    double dscale;       // matrix-core dot products are dscale^-1 times x~.y~ (a power of two; 1 but
                         // for the split FP16 form, whose operands carry a range scale)
    int cost_type;       // COST_* element type of `cost`
    const void* cost;    // METRIC_EXPLICIT: the caller's n x m cost matrix, row-major
};

enum : int { COST_F32 = 0, COST_BF16 = 1, COST_F16 = 2 };

// One cost entry widened exactly to FP32 (a 2-byte entry by its bit pattern).
__device__ __forceinline__ float widen_cost(float v) { return v; }
__device__ __forceinline__ float widen_cost(__bf16 v) {
    return __builtin_bit_cast(float, (uint32_t)__builtin_bit_cast(uint16_t, v) << 16);
}
__device__ __forceinline__ float widen_cost(_Float16 v) { return (float)v; }

// Non-temporal load of one entry of type T, widened to FP32.
template <typename T>
__device__ __forceinline__ float load_cost(const T* p) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_nontemporal_load(p);
    } else {
        const uint16_t bits = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(p));
        return widen_cost(__builtin_bit_cast(T, bits));
    }
}

// The entry at column j of a row: a wave-uniform row base plus a 32-bit byte offset (the
// explicit cost has m <= 2^30 columns), which the loads take as a scalar base and a vector
// offset instead of a 64-bit vector address per load.
template <typename T>
__device__ __forceinline__ float load_cost_col(const T* row, int64_t j) {
    const uint32_t off = (uint32_t)j * (uint32_t)sizeof(T);
    return load_cost(reinterpret_cast<const T*>(reinterpret_cast<const char*>(row) + off));
}

// ---------------------------------------------------------------------------
// Ground costs.  Every kernel works with a pair term P(x, y) defined so that
//     C_ij = s (|x~_i|^2 + |y~_j|^2 - 2 P(x~_i, y~_j)):
// the inner product with the squared norms for the squared Euclidean cost
// (Sections 1 and 4.1), and -dist(x, y)/2 with zero norm arrays for the l1 and
// l_inf costs of the kernelized experiments (Section 5).  The exponent assembly,
// the offsets, the certificate and the cost maximum are then the same for all of them.
// A cost matrix given by the caller (METRIC_EXPLICIT) enters the same way, with
// P_ij = -cost_ij / 2 and zero norms: its points carry index codes instead of
// coordinates (d = 1), row i the code i and column j the code -(j + 1), so that the
// generic pair term finds (i, j) whichever of the two points it is given first.
// ---------------------------------------------------------------------------
enum : int { METRIC_SQEUCLID = 0, METRIC_L1 = 1, METRIC_LINF = 2, METRIC_EXPLICIT = 3 };

// init + P(x, y) with x in registers and y streamed.
template <int M, int D>
__device__ __forceinline__ double pair_term(const double (&x)[D], const double* __restrict__ y, double init) {
    if constexpr (M == METRIC_SQEUCLID) {
        double d = init;
#pragma unroll
        for (int k = 0; k < D; ++k) d = fma(x[k], y[k], d);
        return d;
    } else {
        double a = 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const double t = fabs(x[k] - y[k]);
            a = (M == METRIC_L1) ? a + t : fmax(a, t);
        }
        return fma(-0.5, a, init);
    }
}

// init - cost_ij / 2 for the index codes a, b of a row and a column (either order).
__device__ __forceinline__ double pair_term_cost(const Consts& kc, double a, double b, double init) {
    const bool row_first = a >= 0.0;
    const int64_t i = (int64_t)(row_first ? a : b);
    const int64_t j = -(int64_t)(row_first ? b : a) - 1;
    const int64_t e = i * kc.m + j;
    float v;
    if (kc.cost_type == COST_BF16) v = widen_cost(static_cast<const __bf16*>(kc.cost)[e]);
    else if (kc.cost_type == COST_F16) v = widen_cost(static_cast<const _Float16*>(kc.cost)[e]);
    else v = static_cast<const float*>(kc.cost)[e];
    return fma(-0.5, (double)v, init);
}

// init + P(x, y), both operands in memory, metric and dimension at run time.
__device__ __forceinline__ double pair_term_dyn(const Consts& kc, int D, const double* __restrict__ x,
                                                const double* __restrict__ y, double init) {
    const int M = kc.metric;
    if (M == METRIC_EXPLICIT) return pair_term_cost(kc, x[0], y[0], init);
    if (M == METRIC_SQEUCLID) {
        double d = init;
        for (int k = 0; k < D; ++k) d = fma(x[k], y[k], d);
        return d;
    }
    double a = 0.0;
    for (int k = 0; k < D; ++k) {
        const double t = fabs(x[k] - y[k]);
        a = (M == METRIC_L1) ? a + t : fmax(a, t);
    }
    return fma(-0.5, a, init);
}

// Row data streamed by the column sweep.
struct RowVar {
    double k;   // -sigma^B_i / cfac^B
    float wA;   // r_i 2^(rho sigma^B_i - sigma^A_i)
    float wB;   // r_i
};

__device__ __forceinline__ bool halted(const Ctrl* ctrl) {
    return ctrl->done != 0 || ctrl->t >= ctrl->t_end;
}

__device__ __forceinline__ bool halted_row(const Ctrl* ctrl) {
    return ctrl->done != 0 || ctrl->t_row >= ctrl->t_end;
}

// Sweeps over (blocks of the owned points) x (P splits of the streamed range of length len,
// `split` points each) run on a one-dimensional grid: block b takes split b mod P of owned
// block b / P.  Consecutive block indices go to the eight XCDs in turn, so with P a multiple
// of 8 every XCD streams the same P / 8 splits, whose data then stay in its L2.
struct SweepBlock {
    int64_t bx, p;
};
__device__ __forceinline__ SweepBlock sweep_block(int64_t len, int64_t split) {
    const int64_t P = (len + split - 1) / split;
    return SweepBlock{(int64_t)blockIdx.x / P, (int64_t)blockIdx.x % P};
}

__device__ __forceinline__ float fexp2(double e) {
    return __builtin_amdgcn_exp2f(static_cast<float>(e));
}

// ---------------------------------------------------------------------------
// Preparation: centred FP64 copies, squared norms.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void prep_point(const float* __restrict__ pts, int64_t i, int d,
                                           const float* __restrict__ mu_src_a, const float* __restrict__ mu_src_b,
                                           double* __restrict__ out, double* __restrict__ nrm2,
                                           float* __restrict__ outf, int metric) {
    double acc = 0.0;
    for (int k = 0; k < d; ++k) {
        // centre mu = (x_0 + y_0) / 2: any fixed point works, this one keeps
        // the coordinates of both clouds within one diameter of the origin
        double mu = 0.5 * ((double)mu_src_a[k] + (double)mu_src_b[k]);
        double v = (double)pts[i * d + k] - mu;
        out[i * d + k] = v;
        if (outf) outf[i * d + k] = (float)v;
        acc = fma(v, v, acc);
    }
    nrm2[i] = metric == METRIC_SQEUCLID ? acc : 0.0;   // the l1 / l_inf pair term carries the cost
}

// What the cost maximum starts from: a_j = -|y~_j|^2 / 2 and a cleared result (nullable).
struct MaxStart {
    double* a;
    unsigned long long* bits;
};

// Both clouds in one launch: the n source points, then the m targets.
__global__ void prep_points(const float* __restrict__ x, int64_t n, const float* __restrict__ y, int64_t m, int d,
                            double* __restrict__ xc, double* __restrict__ xn2, float* __restrict__ xcf,
                            double* __restrict__ yc, double* __restrict__ yn2, float* __restrict__ ycf, int metric,
                            MaxStart mx) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e == 0 && mx.bits) *mx.bits = 0ull;
    if (e < n) {
        prep_point(x, e, d, x, y, xc, xn2, xcf, metric);
    } else if (e < n + m) {
        const int64_t j = e - n;
        prep_point(y, j, d, x, y, yc, yn2, ycf, metric);
        if (mx.a) mx.a[j] = -0.5 * yn2[j];
    }
}

// Index codes of the points of an explicit cost matrix: i for row i, -(i + 1) for
// column i; zero norms.
__global__ void prep_cost_codes(int64_t n, int64_t m, double* __restrict__ xc, double* __restrict__ xn2,
                                double* __restrict__ yc, double* __restrict__ yn2, MaxStart mx) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e == 0 && mx.bits) *mx.bits = 0ull;
    if (e < n) {
        xc[e] = (double)e;
        xn2[e] = 0.0;
    } else if (e < n + m) {
        const int64_t j = e - n;
        yc[j] = -(double)(j + 1);
        yn2[j] = 0.0;
        if (mx.a) mx.a[j] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// Column table of iteration t from the state (nu^t, theta^t):
//   g^A_j = -lam_t LOG2E (s yn2_j + K nu_j),  g^B_j = -lam_{t+1} LOG2E (s yn2_j + K nubar_j),
//   nubar = nu + w (theta - nu)  (step:lamp_mid_nu).
// ---------------------------------------------------------------------------
// with offsets != nullptr also a_j = -g^B_j / cfac^B for the exact offsets.  The kernel opens a
// call: the first thread writes the control block if it comes by value (init.write; the schedule
// entry then comes with it) and stops the call before its first iteration (done, err bit 1) if a
// marginal is not a positive vector of sum 1 (init.marginals, from marginal_stats; nullable).
struct CallInit {
    Ctrl ctrl;
    Sched sched;
    const double* marginals;
    int32_t write;
};

__device__ __forceinline__ bool marginals_bad(const double* v) {
    return v[1] >= 0.0 || v[4] >= 0.0 || fabs(v[0] - 1.0) > 1e-9 || fabs(v[3] - 1.0) > 1e-9;
}

__device__ __forceinline__ void col_table_entry(const Consts& kc, const Sched& sc, int64_t t, int64_t j,
                                                const double* __restrict__ yn2, const double* __restrict__ nu,
                                                const double* __restrict__ theta, double2* __restrict__ gtab2,
                                                float2* __restrict__ gtabf, int64_t m_pad,
                                                double* __restrict__ offsets) {
    double nb = nu[j] + sc.w * (theta[j] - nu[j]);
    double base = kc.s * yn2[j];
    double2 g;
    g.x = -sc.lamA * LOG2E * (base + kc.K * nu[j]);
    g.y = -sc.lamB * LOG2E * (base + kc.K * nb);
    gtab2[(t & 1) * kc.m + j] = g;
    if (gtabf) gtabf[(t & 1) * m_pad + j] = make_float2((float)g.x, (float)g.y);
    if (offsets) offsets[j] = -g.y / (2.0 * kc.s * sc.lamB * LOG2E);
}

__global__ void col_table_init(Ctrl* ctrl, Sched* sched, Consts kc, const double* __restrict__ yn2,
                               const double* __restrict__ nu, const double* __restrict__ theta,
                               double2* __restrict__ gtab2, float2* __restrict__ gtabf, int64_t m_pad,
                               double* __restrict__ offsets, CallInit init) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t t = init.write ? init.ctrl.t : ctrl->t;
    const Sched sc = init.write ? init.sched : sched[t - ctrl->t_base];
    if (j == 0) {
        if (init.write) {
            *ctrl = init.ctrl;
            sched[0] = init.sched;
        }
        if (init.marginals && marginals_bad(init.marginals)) {
            ctrl->done = 1;
            ctrl->done_seen = 1;
            ctrl->err = 2;
        }
    }
    if (j < kc.m) col_table_entry(kc, sc, t, j, yn2, nu, theta, gtab2, gtabf, m_pad, offsets);
}

// The iterate of the workspace's buffers into the caller's state, unless the call was stopped by
// its marginals.
__global__ void commit_state(const Ctrl* ctrl, int64_t m, const double* __restrict__ nu1,
                             const double* __restrict__ th1, double* __restrict__ nu, double* __restrict__ theta) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m || (ctrl->err & 2)) return;
    nu[j] = nu1[j];
    theta[j] = th1[j];
}

// ---------------------------------------------------------------------------
// Row extreme sweep: out_i = min_j (a_j + sgn * x~_i . y~_j), FP64, exact.
// Used for the exact offsets, D(theta) and the cost maximum.
// part: [P][n] partial minima over column splits.
// ---------------------------------------------------------------------------
template <int M, int D>
__device__ __forceinline__ void row_extreme_body(Consts kc, const double* __restrict__ xc,
                                                     const double* __restrict__ yc,
                                                     const double* __restrict__ a, double sgn,
                                                     double* __restrict__ part, int64_t split, int64_t bx_, int64_t by_, int64_t nb_) {
    const int64_t i = (int64_t)bx_ * BLOCK + threadIdx.x;
    const int64_t p = by_;
    const int64_t j0 = p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double x[D];
    // a_j + sgn P(x_i, y_j): the inner product takes the sign on x and starts from a_j, the
    // distances, and the dimensions 9 to 15, take both after (the order of the run-time form,
    // which an offset shares to the last bit: a trajectory keeps its FP32 roundings)
    constexpr bool FROM_A = M == METRIC_SQEUCLID && (D <= 8 || D == 16);
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = (FROM_A ? sgn : 1.0) * xc[ii * D + k];
    auto term = [&](const double* yj, double aj) {
        return FROM_A ? pair_term<M, D>(x, yj, aj) : fma(sgn, pair_term<M, D>(x, yj, 0.0), aj);
    };
    // blocks of UNROLL columns with independent chains, as in the sweeps: the column data
    // are wave-uniform and their scalar loads overlap the arithmetic of the block
    double best = __builtin_inf();
    const int nfull = (int)((j1 - j0) / UNROLL);
    const double* __restrict__ yp = yc + j0 * D;
    const double* __restrict__ ap = a + j0;
    for (int c = 0; c < nfull; ++c, yp += UNROLL * D, ap += UNROLL) {
        double v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = term(yp + u * D, ap[u]);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) best = fmin(best, v[u]);
    }
    const int rem = (int)((j1 - j0) - (int64_t)nfull * UNROLL);
    for (int u = 0; u < rem; ++u) best = fmin(best, term(yp + u * D, ap[u]));
    if (i < kc.n) part[p * kc.n + i] = best;
}

template <int M, int D>
__global__ __launch_bounds__(BLOCK) void row_extreme(Consts kc, const double* __restrict__ xc,
                                                     const double* __restrict__ yc,
                                                     const double* __restrict__ a, double sgn,
                                                     double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    row_extreme_body<M, D>(kc, xc, yc, a, sgn, part, split, sb.bx, sb.p, 0);
}

// Generic-d version: coordinates read per pair.
__device__ __forceinline__ void row_extreme_dyn_body(Consts kc, int D, const double* __restrict__ xc,
                                                         const double* __restrict__ yc,
                                                         const double* __restrict__ a, double sgn,
                                                         double* __restrict__ part, int64_t split, int64_t bx_, int64_t by_, int64_t nb_) {
    const int64_t i = (int64_t)bx_ * BLOCK + threadIdx.x;
    const int64_t p = by_;
    const int64_t j0 = p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double best = __builtin_inf();
    for (int64_t j = j0; j < j1; ++j) {
        best = fmin(best, fma(sgn, pair_term_dyn(kc, D, xc + ii * D, yc + j * D, 0.0), a[j]));
    }
    if (i < kc.n) part[p * kc.n + i] = best;
}

__global__ __launch_bounds__(BLOCK) void row_extreme_dyn(Consts kc, int D, const double* __restrict__ xc,
                                                         const double* __restrict__ yc,
                                                         const double* __restrict__ a, double sgn,
                                                         double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    row_extreme_dyn_body(kc, D, xc, yc, a, sgn, part, split, sb.bx, sb.p, 0);
}

// The least of the partial minima of row i (exact, order independent).
__device__ __forceinline__ double merge_minima(const double* __restrict__ part, int P, int64_t n, int64_t i) {
    double best = part[i];
#pragma unroll 8
    for (int p = 1; p < P; ++p) best = fmin(best, part[(int64_t)p * n + i]);
    return best;
}

__global__ void row_extreme_merge(Consts kc, const double* __restrict__ part, int P, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kc.n) out[i] = merge_minima(part, P, kc.n, i);
}

// The largest xn2_i - 2 min_i over the rows into *bits (cleared before), and each row's value if
// rowmax is given.  Non-negative doubles order as their bits do; a NaN counts as 0, and so does a
// negative rounding of 0.
__device__ __forceinline__ void row_extreme_max_body(int64_t n, const double* __restrict__ part, int P,
                                                     const double* __restrict__ xn2, double* __restrict__ rowmax,
                                                     unsigned long long* __restrict__ bits, int64_t i) {
    double v = 0.0;
    if (i < n) {
        const double row = xn2[i] - 2.0 * merge_minima(part, P, n, i);
        if (rowmax) rowmax[i] = row;
        v = fmax(row, 0.0);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0 && v > 0.0) atomicMax(bits, (unsigned long long)__double_as_longlong(v));
}

__global__ void row_extreme_max(Consts kc, const double* __restrict__ part, int P, const double* __restrict__ xn2,
                                double* __restrict__ rowmax, unsigned long long* __restrict__ bits) {
    row_extreme_max_body(kc.n, part, P, xn2, rowmax, bits, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// ---------------------------------------------------------------------------
// Row sweep: the two row sums S^A_i, S^B_i with the shared offset h_i.
// part: [P][n] double2.
// ---------------------------------------------------------------------------
// e = a * b + c with c wave-uniform (an SGPR pair).  The VOP3 form takes the
// scalar operand directly; the compiler otherwise copies c into VGPRs for the
// two-address v_fmac_f64 form, costing two extra VALU moves per use.
__device__ __forceinline__ double fma_su(double a, double b, double c_uniform) {
    double e;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(e) : "v"(a), "v"(b), "s"(c_uniform));
    return e;
}

// Streamed points whose scalar loads are in flight together: from D = 9 on two.  The coordinates of all
// UNROLL points do not fit the scalar registers there, and the compiler, loading them all the same,
// moved them through vector lanes (48 of 244 vector instructions a group at D = 16): 20011 x 20011
// column sweep at D = 16 382 -> 310 us, 12 256 -> 248; 40 problems at D = 16 in a batch 39.4 -> 32.6 ms.
// Up to D = 8 the fence costs 1 to 2% (D = 6 183 -> 186 us).  TIGHT: for a kernel that holds more
// scalars beside the loop, the most points whose coordinates and pair of exponent terms fit 64.
template <int D, bool TIGHT>
constexpr int loads_together() {
    if (!TIGHT) return D <= 8 ? UNROLL : 2;
    return D <= 2 ? UNROLL : D <= 6 ? 4 : 2;
}

template <int D, bool TIGHT = false>
__device__ __forceinline__ void loads_fence(int u) {
    if (u % loads_together<D, TIGHT>() == 0 && u > 0) __builtin_amdgcn_sched_barrier(0);
}

// One column j of the row sweep for this lane's row: returns 2^eA, 2^eB.
template <int M, int D>
__device__ __forceinline__ void row_terms(const double (&x)[D], double h, const double* __restrict__ yj,
                                          double2 g, double cA, double cB, float& pA, float& pB) {
    const double dot = pair_term<M, D>(x, yj, h);
    pA = fexp2(fma_su(dot, cA, g.x));
    pB = fexp2(fma_su(dot, cB, g.y));
}

// The same with the cost term of the B coupling for D_t tracking: tB = 2^eB C_ij / s, with
// C_ij / s = |x~_i|^2 + |y~_j|^2 - 2 P_ij taken from the exponent's dot product
// dot = h + P_ij as (|x~_i|^2 + 2 h + |y~_j|^2) - 2 dot (xa = |x~_i|^2 + 2 h; the norms are
// zero for l1 / l_inf, where P_ij = -dist / 2): two FP64 operations, a conversion and an FMA.
template <int M, int D>
__device__ __forceinline__ void row_terms_dt(const double (&x)[D], double h, double xa, const double* __restrict__ yj,
                                             double yn2j, double2 g, double cA, double cB, float& pA, float& pB,
                                             float& tB) {
    const double dot = pair_term<M, D>(x, yj, h);
    pA = fexp2(fma_su(dot, cA, g.x));
    pB = fexp2(fma_su(dot, cB, g.y));
    const double cs = fma(-2.0, dot, M == METRIC_SQEUCLID ? xa + yn2j : xa);
    tB = pB * (float)cs;
}

// The row sums of one lane's row over the columns [j0, j1).
template <int M, int D, bool TIGHT = false>
__device__ __forceinline__ void row_sweep_run(double cA, double cB, const double (&x)[D], double h,
                                              const double* __restrict__ yc, const double2* __restrict__ g,
                                              int64_t j0, int64_t j1, double& sumA, double& sumB) {
    const int nfull = (int)((j1 - j0) / UNROLL);
    const double* __restrict__ yp = yc + j0 * D;
    const double2* __restrict__ gp = g + j0;
    for (int c = 0; c < nfull; ++c, yp += UNROLL * D, gp += UNROLL) {
        float pA[UNROLL], pB[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            loads_fence<D, TIGHT>(u);
            row_terms<M, D>(x, h, yp + u * D, gp[u], cA, cB, pA[u], pB[u]);
        }
        float accA = pA[0], accB = pB[0];
#pragma unroll
        for (int u = 1; u < UNROLL; ++u) {
            accA += pA[u];
            accB += pB[u];
        }
        sumA += (double)accA;
        sumB += (double)accB;
    }
    const int rem = (int)((j1 - j0) - (int64_t)nfull * UNROLL);
    float accA = 0.f, accB = 0.f;
    for (int u = 0; u < rem; ++u) {
        float a, b;
        row_terms<M, D>(x, h, yp + u * D, gp[u], cA, cB, a, b);
        accA += a;
        accB += b;
    }
    sumA += (double)accA;
    sumB += (double)accB;
}

// Row sweep body; with DT the sweep also sums the B coupling's cost terms for D_t tracking
// (tpart[p][i], under the same row offset as the B sums, so the splits add up directly).
template <int M, int D, bool DT = false>
__device__ __forceinline__ void row_sweep_body(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                   const double* __restrict__ xc,
                                                   const double* __restrict__ yc,
                                                   const double2* __restrict__ gtab2,
                                                   const double* __restrict__ H,
                                                   double2* __restrict__ part, int64_t split, int64_t bx_, int64_t by_, int64_t nb_,
                                                   const double* __restrict__ xn2 = nullptr,
                                                   const double* __restrict__ yn2 = nullptr,
                                                   double* __restrict__ tpart = nullptr) {
    if (halted_row(ctrl)) return;
    const int64_t t = ctrl->t_row;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const double2* __restrict__ g = gtab2 + (t & 1) * kc.m;

    const int64_t i = (int64_t)bx_ * BLOCK + threadIdx.x;
    const int64_t p = by_;
    const int64_t j0 = p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double x[D];
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = xc[ii * D + k];
    const double h = H[ii];

    double sumA = 0.0, sumB = 0.0, sumT = 0.0;
    if constexpr (!DT) {
        row_sweep_run<M, D>(cA, cB, x, h, yc, g, j0, j1, sumA, sumB);
    } else {
        const double xa = (M == METRIC_SQEUCLID ? xn2[ii] : 0.0) + 2.0 * h;
        // pointers that step, and the two couplings' sums before the cost's: 2.30 ms a sweep at 65536 x 65536 x 3,
        // 2.50 with an index and all three side by side
        const int nfull = (int)((j1 - j0) / UNROLL);
        const double* __restrict__ yp = yc + j0 * D;
        const double2* __restrict__ gp = g + j0;
        const double* __restrict__ np = yn2 + j0;
        for (int c = 0; c < nfull; ++c, yp += UNROLL * D, gp += UNROLL, np += UNROLL) {
            float pA[UNROLL], pB[UNROLL], tB[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                row_terms_dt<M, D>(x, h, xa, yp + u * D, M == METRIC_SQEUCLID ? np[u] : 0.0, gp[u], cA, cB, pA[u],
                                   pB[u], tB[u]);
            float accA = pA[0], accB = pB[0], accT = tB[0];
#pragma unroll
            for (int u = 1; u < UNROLL; ++u) {
                accA += pA[u];
                accB += pB[u];
            }
            sumA += (double)accA;
            sumB += (double)accB;
#pragma unroll
            for (int u = 1; u < UNROLL; ++u) accT += tB[u];
            sumT += (double)accT;
        }
        const int rem = (int)((j1 - j0) - (int64_t)nfull * UNROLL);
        float accA = 0.f, accB = 0.f, accT = 0.f;
        for (int u = 0; u < rem; ++u) {
            float a, b, tb;
            row_terms_dt<M, D>(x, h, xa, yp + u * D, M == METRIC_SQEUCLID ? np[u] : 0.0, gp[u], cA, cB, a, b, tb);
            accA += a;
            accB += b;
            accT += tb;
        }
        sumA += (double)accA;
        sumB += (double)accB;
        sumT += (double)accT;
    }
    if (i < kc.n) {
        part[p * kc.n + i] = make_double2(sumA, sumB);
        if constexpr (DT) tpart[p * kc.n + i] = sumT;
    }
}

template <int M, int D>
__global__ __launch_bounds__(BLOCK) void row_sweep(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                   const double* __restrict__ xc,
                                                   const double* __restrict__ yc,
                                                   const double2* __restrict__ gtab2,
                                                   const double* __restrict__ H,
                                                   double2* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    row_sweep_body<M, D>(ctrl, sched, kc, xc, yc, gtab2, H, part, split, sb.bx, sb.p, 0);
}

// Column groups of a split summed in parallel by the waves of a block (see row_sweep_par).
__device__ __forceinline__ float* group_sums() {
    extern __shared__ __align__(16) float lds_group_sums[];
    return lds_group_sums;
}

// The FP64 sums of a split from its FP32 group sums in LDS ([2][groups][64]), in group order: the
// first two waves of the block take one coupling each.
__device__ __forceinline__ double sum_groups(const float* sums, int groups, int lane) {
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < groups; ++c) s += (double)sums[c * 64 + lane];
    return s;
}

// Row sweep for grids that leave the chip short of waves: a block owns 64 rows of a split and its
// waves share the split's groups of UNROLL columns; the group sums meet in LDS and are added in
// the order of row_sweep, so that the results are the same to the last bit.
template <int M, int D>
__global__ __launch_bounds__(1024) void row_sweep_par(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                      const double* __restrict__ xc, const double* __restrict__ yc,
                                                      const double2* __restrict__ gtab2,
                                                      const double* __restrict__ H, double2* __restrict__ part,
                                                      int64_t split) {
    if (halted_row(ctrl)) return;
    const int64_t t = ctrl->t_row;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const double2* __restrict__ g = gtab2 + (t & 1) * kc.m;
    const SweepBlock sb = sweep_block(kc.m, split);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int64_t i = sb.bx * 64 + lane;
    const int64_t j0 = sb.p * split;
    const int len = (int)(min(kc.m, j0 + split) - j0);
    const int groups = (len + UNROLL - 1) / UNROLL;
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double x[D];
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = xc[ii * D + k];
    const double h = H[ii];
    float* sums = group_sums();
    const int c1 = (wave + 1) * groups / waves;
    for (int c = wave * groups / waves; c < c1; ++c) {
        const double* __restrict__ yp = yc + (j0 + c * UNROLL) * D;
        const double2* __restrict__ gp = g + j0 + c * UNROLL;
        float accA = 0.f, accB = 0.f;
        if ((c + 1) * UNROLL <= len) {
            float pA[UNROLL], pB[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                loads_fence<D>(u);
                row_terms<M, D>(x, h, yp + u * D, gp[u], cA, cB, pA[u], pB[u]);
            }
            accA = pA[0];
            accB = pB[0];
#pragma unroll
            for (int u = 1; u < UNROLL; ++u) {
                accA += pA[u];
                accB += pB[u];
            }
        } else {
            for (int u = 0; u < len - c * UNROLL; ++u) {
                float a, b;
                row_terms<M, D>(x, h, yp + u * D, gp[u], cA, cB, a, b);
                accA += a;
                accB += b;
            }
        }
        sums[c * 64 + lane] = accA;
        sums[(groups + c) * 64 + lane] = accB;
    }
    __syncthreads();
    if (wave < 2 && i < kc.n)
        reinterpret_cast<double*>(part)[2 * (sb.p * kc.n + i) + wave] = sum_groups(sums + wave * groups * 64, groups, lane);
}

// The row sweep of a D_t-tracked iteration: the row sweep above plus the B coupling's cost
// sums, tpart: [P][n].
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void row_sweep_dt(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                      const double* __restrict__ xc,
                                                      const double* __restrict__ yc,
                                                      const double2* __restrict__ gtab2,
                                                      const double* __restrict__ H,
                                                      double2* __restrict__ part, int64_t split,
                                                      const double* __restrict__ xn2,
                                                      const double* __restrict__ yn2,
                                                      double* __restrict__ tpart) {
    const SweepBlock sb = sweep_block(kc.m, split);
    row_sweep_body<M, D, true>(ctrl, sched, kc, xc, yc, gtab2, H, part, split, sb.bx, sb.p, 0, xn2, yn2, tpart);
}

// The row sums of one lane's row, at xi, for a run-time dimension.
__device__ __forceinline__ void row_sweep_run_dyn(const Consts& kc, int D, double cA, double cB,
                                                  const double* __restrict__ xi, double h,
                                                  const double* __restrict__ yc, const double2* __restrict__ g,
                                                  int64_t j0, int64_t j1, double& sumA, double& sumB) {
    for (int64_t jb = j0; jb < j1; jb += UNROLL) {
        float accA = 0.f, accB = 0.f;
        const int64_t je = min(j1, jb + UNROLL);
        for (int64_t j = jb; j < je; ++j) {
            const double dot = pair_term_dyn(kc, D, xi, yc + j * D, h);
            accA += fexp2(fma(cA, dot, g[j].x));
            accB += fexp2(fma(cB, dot, g[j].y));
        }
        sumA += (double)accA;
        sumB += (double)accB;
    }
}

__global__ __launch_bounds__(BLOCK) void row_sweep_dyn(const Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                                                       const double* __restrict__ xc,
                                                       const double* __restrict__ yc,
                                                       const double2* __restrict__ gtab2,
                                                       const double* __restrict__ H,
                                                       double2* __restrict__ part, int64_t split) {
    if (halted_row(ctrl)) return;
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t t = ctrl->t_row;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    const int64_t j0 = sb.p * split;
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double sumA = 0.0, sumB = 0.0;
    row_sweep_run_dyn(kc, D, cA, cB, xc + ii * D, H[ii], yc, gtab2 + (t & 1) * kc.m, j0, min(kc.m, j0 + split), sumA,
                      sumB);
    if (i < kc.n) part[sb.p * kc.n + i] = make_double2(sumA, sumB);
}

// Exact recomputation of sigma_i = log2 sum_j 2^(g_j + cfac x~_i.y~_j) (two passes, FP64 max).
__device__ double exact_sigma(const Consts& kc, const double* __restrict__ xi, const double* __restrict__ yc, int D,
                              const double2* __restrict__ g, int which, double cfac) {
    const int64_t m = kc.m;
    double mx = -__builtin_inf();
    for (int64_t j = 0; j < m; ++j) {
        const double dot = pair_term_dyn(kc, D, xi, yc + j * D, 0.0);
        double e = fma(cfac, dot, which ? g[j].y : g[j].x);
        mx = fmax(mx, e);
    }
    double s = 0.0;
    for (int64_t j = 0; j < m; ++j) {
        const double dot = pair_term_dyn(kc, D, xi, yc + j * D, 0.0);
        double e = fma(cfac, dot, which ? g[j].y : g[j].x);
        s += exp2(e - mx);
    }
    return mx + log2(s);
}

// The sums over the splits, in split order, from the partials of point i ([P][len]): blocks of 32
// and 8 independent loads (a merge is bound by the latency of its loads: with 8 in flight at most
// 32 splits of 4096 rows took 4.6 us).
__device__ __forceinline__ double2 merge_splits(const double2* __restrict__ part, int P, int64_t len, int64_t i) {
    double a = 0.0, b = 0.0;
    int p = 0;
    auto take = [&](auto cnt) {
        constexpr int U = decltype(cnt)::value;
        double2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = part[(int64_t)(p + u) * len + i];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a += v[u].x;
            b += v[u].y;
        }
        p += U;
    };
    while (p + 32 <= P) take(std::integral_constant<int, 32>{});
    while (p + 8 <= P) take(std::integral_constant<int, 8>{});
    while (p < P) take(std::integral_constant<int, 1>{});
    return make_double2(a, b);
}

// Merge the row partials; derive sigma^A, sigma^B, the next offsets and the
// column-sweep row data; optional natural-log normalisers.
// FP32 row data of the matrix-core column sweep (nullable): {k, w^A, w^B, 0} per row,
// k rounded to FP32 with the rounding error folded exactly into the weights.
// f32_offsets: the row sweep applied (float)H, so that value is the one to subtract.
struct RowVarF32 {
    float4* q;
    int f32_offsets;
};

__device__ __forceinline__ void row_finish_body(Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                           const double* __restrict__ xc, const double* __restrict__ yc,
                           const double2* __restrict__ gtab2, const double* __restrict__ r,
                           const double* __restrict__ xn2, const double2* __restrict__ part, int P,
                           double* __restrict__ H, RowVar* __restrict__ rowvar, double2* __restrict__ rowck,
                           double* __restrict__ log_za, double* __restrict__ log_zb, RowVarF32 rf, int32_t done, int64_t bx_) {
    if (done || ctrl->err || ctrl->t_row >= ctrl->t_end) return;
    int64_t i = (int64_t)bx_ * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t t = ctrl->t_row;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const double2 S = merge_splits(part, P, kc.n, i);
    const double SA = S.x, SB = S.y;
    const double h = rf.f32_offsets ? (double)(float)H[i] : H[i];
    double sigA, sigB;
    const double lo = 0x1p-60, hi = 0x1p+60;
    if (SA >= lo && SA <= hi && SB >= lo && SB <= hi) {
        sigA = log2(SA) - cA * h;
        sigB = log2(SB) - cB * h;
    } else {
        const double2* g = gtab2 + (t & 1) * kc.m;
        sigA = exact_sigma(kc, xc + i * D, yc, D, g, 0, cA);
        sigB = exact_sigma(kc, xc + i * D, yc, D, g, 1, cB);
        atomicAdd(&ctrl->fallbacks_row, 1);
    }
    const double hnew = -sigB / cB;
    const double rho = cA / cB;
    double ew = rho * sigB - sigA;
    ew = fmin(fmax(ew, -1000.0), 1000.0);
    H[i] = hnew;
    // The column sweeps that take FP32 row weights see the A factor 2^ew in w^A; a row with
    // |ew| > 100 (large tau1: ew grows with K tau1 (theta - nu)) moves their shared offset by
    // dl = ew / (c^A + c^B), which leaves |ew| / (1 + rho) in each weight's exponent
    // (w^A 2^(c^A (x.y + k)) and w^B 2^(c^B (x.y + k)) are unchanged).
    double kw = hnew, ea = ew, eb = 0.0;
    if (fabs(ew) > 100.0) {
        const double dl = ew / (cA + cB);
        kw = hnew + dl;
        ea = ew - cA * dl;
        eb = -cB * dl;
    }
    RowVar rv;
    rv.k = kw;
    rv.wA = (float)(r[i] * exp2(ea));
    rv.wB = (float)(r[i] * exp2(eb));
    rowvar[i] = rv;
    // the vector-ALU column sweep takes the row weights into its exponents: the A coupling's
    // row factor 2^ew (unclamped: no FP32 weight to overflow) and n r_i (1 for uniform r; the
    // sweep multiplies its sums by 1/n)
    if (rowck) {
        const double lw = log2((double)kc.n * r[i]);
        rowck[i] = make_double2(cA * hnew + (rho * sigB - sigA) + lw, cB * hnew + lw);
    }
    if (rf.q) {
        const float kf = (float)kw;
        const double dk = kw - (double)kf;
        const float wa = (float)(r[i] * exp2(fmin(fmax(ea + cA * dk, -1000.0), 1000.0)));
        const float wb = (float)(r[i] * exp2(eb + cB * dk));
        rf.q[i] = make_float4(kf, wa, wb, 0.f);
    }
    if (log_za) log_za[i] = LN2 * (-sc.lamA * LOG2E * kc.s * xn2[i] + sigA);
    if (log_zb) log_zb[i] = LN2 * (-sc.lamB * LOG2E * kc.s * xn2[i] + sigB);
}

// ---------------------------------------------------------------------------
// Column sweep: col^A_j, col^B_j.  cpart: [P][m] double2.
// ---------------------------------------------------------------------------
// One row i of the column sweep for this lane's column.  With k_i the row's offset,
// ew_i = rho sigma^B_i - sigma^A_i the A coupling's row factor and G_j = g^B_j / cfac^B this
// column's term, the base-2 exponents of the normalised couplings are
//     e^B = cfac^B (P_ij + G_j) + cfac^B k_i,
//     e^A = cfac^A (P_ij + G_j) + (cfac^A k_i + ew_i) + D_j,   D_j = g^A_j - cfac^A G_j:
// the dot product starts from G_j (per lane), the row terms come precomputed (rowck,
// scalar, with the row weight as log2(n r_i) in both), and D_j, constant down the column,
// is applied once to the column's A sum (`factor`) or added to each exponent; the sums are
// plain FP32 adds, multiplied by 1/n at the end.
template <int M, int D, bool FACTOR>
__device__ __forceinline__ void col_terms(const double (&y)[D], const double* __restrict__ xi, double2 ck,
                                          double G, double Dj, double cA, double cB, float& accA, float& accB) {
    const double dot = pair_term<M, D>(y, xi, G);   // the distances are symmetric
    double eA = fma_su(dot, cA, ck.x);
    if constexpr (!FACTOR) eA += Dj;
    accA += fexp2(eA);
    accB += fexp2(fma_su(dot, cB, ck.y));
}

template <int M, int D, bool FACTOR, bool TIGHT = false>
__device__ __forceinline__ void col_sweep_run(double cA, double cB, const double (&y)[D], double G, double Dj,
                                              const double* __restrict__ xc, const double2* __restrict__ rowck,
                                              int64_t i0, int64_t i1, double& sumA, double& sumB) {
    const int nfull = (int)((i1 - i0) / UNROLL);
    const double* __restrict__ xp = xc + i0 * D;
    const double2* __restrict__ kp = rowck + i0;
    for (int c = 0; c < nfull; ++c, xp += UNROLL * D, kp += UNROLL) {
        float accA = 0.f, accB = 0.f;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            loads_fence<D, TIGHT>(u);
            col_terms<M, D, FACTOR>(y, xp + u * D, kp[u], G, Dj, cA, cB, accA, accB);
        }
        sumA += (double)accA;
        sumB += (double)accB;
    }
    const int rem = (int)((i1 - i0) - (int64_t)nfull * UNROLL);
    float accA = 0.f, accB = 0.f;
    for (int u = 0; u < rem; ++u) col_terms<M, D, FACTOR>(y, xp + u * D, kp[u], G, Dj, cA, cB, accA, accB);
    sumA += (double)accA;
    sumB += (double)accB;
}

template <int M, int D>
__device__ __forceinline__ void col_sweep_body(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                   const double* __restrict__ xc,
                                                   const double* __restrict__ yc,
                                                   const double2* __restrict__ gtab2,
                                                   const RowVar* __restrict__ rowvar,
                                                   const double2* __restrict__ rowck,
                                                   double2* __restrict__ cpart, int64_t split, int64_t bx_, int64_t by_, int64_t nb_) {
    if (halted(ctrl)) return;
    const int64_t t = ctrl->t;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const int64_t j = (int64_t)bx_ * BLOCK + threadIdx.x;
    const int64_t p = by_;
    const int64_t i0 = p * split;
    const int64_t i1 = min(kc.n, i0 + split);
    const int64_t jj = j < kc.m ? j : kc.m - 1;
    double y[D];
#pragma unroll
    for (int k = 0; k < D; ++k) y[k] = yc[jj * D + k];
    const double2 g = gtab2[(t & 1) * kc.m + jj];
    const double G = g.y / cB;
    const double Dj = g.x - cA * G;

    double sumA = 0.0, sumB = 0.0;
    const double inv_n = 1.0 / (double)kc.n;   // the row weights r_i enter as n r_i (rowck)
    if (kc.factor_cols) {
        col_sweep_run<M, D, true>(cA, cB, y, G, Dj, xc, rowck, i0, i1, sumA, sumB);
        sumA *= exp2(Dj) * inv_n;
    } else {
        col_sweep_run<M, D, false>(cA, cB, y, G, Dj, xc, rowck, i0, i1, sumA, sumB);
        sumA *= inv_n;
    }
    sumB *= inv_n;
    if (j < kc.m) cpart[p * kc.m + j] = make_double2(sumA, sumB);
}

template <int M, int D>
__global__ __launch_bounds__(BLOCK) void col_sweep(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                   const double* __restrict__ xc,
                                                   const double* __restrict__ yc,
                                                   const double2* __restrict__ gtab2,
                                                   const RowVar* __restrict__ rowvar,
                                                   const double2* __restrict__ rowck,
                                                   double2* __restrict__ cpart, int64_t split) {
    const SweepBlock sb = sweep_block(kc.n, split);
    col_sweep_body<M, D>(ctrl, sched, kc, xc, yc, gtab2, rowvar, rowck, cpart, split, sb.bx, sb.p, 0);
}

// Column sweep for grids that leave the chip short of waves, as row_sweep_par.
template <int M, int D>
__global__ __launch_bounds__(1024) void col_sweep_par(const Ctrl* ctrl, const Sched* sched, Consts kc,
                                                      const double* __restrict__ xc, const double* __restrict__ yc,
                                                      const double2* __restrict__ gtab2,
                                                      const double2* __restrict__ rowck,
                                                      double2* __restrict__ cpart, int64_t split) {
    if (halted(ctrl)) return;
    const int64_t t = ctrl->t;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const SweepBlock sb = sweep_block(kc.n, split);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int64_t j = sb.bx * 64 + lane;
    const int64_t i0 = sb.p * split;
    const int len = (int)(min(kc.n, i0 + split) - i0);
    const int groups = (len + UNROLL - 1) / UNROLL;
    const int64_t jj = j < kc.m ? j : kc.m - 1;
    double y[D];
#pragma unroll
    for (int k = 0; k < D; ++k) y[k] = yc[jj * D + k];
    const double2 g = gtab2[(t & 1) * kc.m + jj];
    const double G = g.y / cB;
    const double Dj = g.x - cA * G;
    float* sums = group_sums();
    auto run = [&](auto factor) {
        constexpr bool FACTOR = decltype(factor)::value;
        const int c1 = (wave + 1) * groups / waves;
        for (int c = wave * groups / waves; c < c1; ++c) {
            const double* __restrict__ xp = xc + (i0 + c * UNROLL) * D;
            const double2* __restrict__ kp = rowck + i0 + c * UNROLL;
            float accA = 0.f, accB = 0.f;
            if ((c + 1) * UNROLL <= len) {
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    loads_fence<D>(u);
                    col_terms<M, D, FACTOR>(y, xp + u * D, kp[u], G, Dj, cA, cB, accA, accB);
                }
            } else {
                for (int u = 0; u < len - c * UNROLL; ++u)
                    col_terms<M, D, FACTOR>(y, xp + u * D, kp[u], G, Dj, cA, cB, accA, accB);
            }
            sums[c * 64 + lane] = accA;
            sums[(groups + c) * 64 + lane] = accB;
        }
    };
    if (kc.factor_cols) run(std::true_type{});
    else run(std::false_type{});
    __syncthreads();
    if (wave < 2 && j < kc.m) {
        const double inv_n = 1.0 / (double)kc.n;   // the row weights r_i enter as n r_i (rowck)
        double s = sum_groups(sums + wave * groups * 64, groups, lane);
        s *= wave == 0 && kc.factor_cols ? exp2(Dj) * inv_n : inv_n;
        reinterpret_cast<double*>(cpart)[2 * (sb.p * kc.m + j) + wave] = s;
    }
}

// The column sums of one lane's column, at yj, for a run-time dimension (the exponent assembly of col_terms).
__device__ __forceinline__ void col_sweep_run_dyn(const Consts& kc, int D, double cA, double cB,
                                                  const double* __restrict__ yj, double G, double Dj,
                                                  const double* __restrict__ xc, const double2* __restrict__ rowck,
                                                  int64_t i0, int64_t i1, double& sumA, double& sumB) {
    for (int64_t ib = i0; ib < i1; ib += UNROLL) {
        float accA = 0.f, accB = 0.f;
        const int64_t ie = min(i1, ib + UNROLL);
        for (int64_t i = ib; i < ie; ++i) {
            const double2 ck = rowck[i];
            const double dot = pair_term_dyn(kc, D, yj, xc + i * D, G);
            double eA = fma(dot, cA, ck.x);
            if (!kc.factor_cols) eA += Dj;
            accA += fexp2(eA);
            accB += fexp2(fma(dot, cB, ck.y));
        }
        sumA += (double)accA;
        sumB += (double)accB;
    }
}

__global__ __launch_bounds__(BLOCK) void col_sweep_dyn(const Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                                                       const double* __restrict__ xc,
                                                       const double* __restrict__ yc,
                                                       const double2* __restrict__ gtab2,
                                                       const RowVar* __restrict__ rowvar,
                                                       const double2* __restrict__ rowck,
                                                       double2* __restrict__ cpart, int64_t split) {
    if (halted(ctrl)) return;
    const SweepBlock sb = sweep_block(kc.n, split);
    const int64_t t = ctrl->t;
    const Sched sc = sched[t - ctrl->t_base];
    const double cA = 2.0 * kc.s * sc.lamA * LOG2E;
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const int64_t j = sb.bx * BLOCK + threadIdx.x;
    const int64_t i0 = sb.p * split;
    const int64_t jj = j < kc.m ? j : kc.m - 1;
    const double2 g = gtab2[(t & 1) * kc.m + jj];
    const double G = g.y / cB;
    const double Dj = g.x - cA * G;
    double sumA = 0.0, sumB = 0.0;
    col_sweep_run_dyn(kc, D, cA, cB, yc + jj * D, G, Dj, xc, rowck, i0, min(kc.n, i0 + split), sumA, sumB);
    const double inv_n = 1.0 / (double)kc.n;
    sumA *= (kc.factor_cols ? exp2(Dj) : 1.0) * inv_n;
    sumB *= inv_n;
    if (j < kc.m) cpart[sb.p * kc.m + j] = make_double2(sumA, sumB);
}

// ---------------------------------------------------------------------------
// D_t tracking (Proposition infeas_bound(b)): <C, Xbar^{t+1}> of the second coupling
// of iteration t, Xbar^{t+1} = diag(r) p^{eta_{t+1}}(nubar^{t+1}).  Per row, with the
// row sweep's offset h_i and column table g^B:
//     S_i = sum_j 2^(cB (h_i + P_ij) + g^B_j),   T_i = sum_j 2^(...) C_ij,
//     out_i = r_i T_i / S_i  (the normaliser cancels),  C_ij = s (|x~_i|^2 + |y~_j|^2 - 2 P_ij).
// Same arithmetic as the row sweep (FP64 exponent, FP32 exponential and per-block
// sums, FP64 across blocks); one thread per row over all columns.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void dt_cost_rows_dyn(const Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                                                          const double* __restrict__ xc,
                                                          const double* __restrict__ yc,
                                                          const double* __restrict__ xn2,
                                                          const double* __restrict__ yn2,
                                                          const double2* __restrict__ gtab2,
                                                          const double* __restrict__ H,
                                                          const double* __restrict__ r,
                                                          double* __restrict__ out) {
    if (halted(ctrl)) return;
    const int64_t t = ctrl->t;
    const Sched sc = sched[t - ctrl->t_base];
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const double2* __restrict__ g = gtab2 + (t & 1) * kc.m;
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    const double h = H[ii];
    const double xa = kc.s * xn2[ii];
    double S = 0.0, T = 0.0;
    for (int64_t jb = 0; jb < kc.m; jb += UNROLL) {
        float aS = 0.f, aT = 0.f;
        const int64_t je = min(kc.m, jb + UNROLL);
        for (int64_t j = jb; j < je; ++j) {
            const double dot = pair_term_dyn(kc, D, xc + ii * D, yc + j * D, 0.0);
            const float p = fexp2(fma(cB, h + dot, g[j].y));
            const double cij = fma(-2.0 * kc.s, dot, xa + kc.s * yn2[j]);
            aS += p;
            aT = fmaf(p, (float)cij, aT);
        }
        S += (double)aS;
        T += (double)aT;
    }
    if (i < kc.n) out[i] = r[i] * T / S;
}

// Row i's share of <C, Xbar^{t+1}> from the D_t-tracked row sweep's splits: s r_i T_i / S^B_i
// (both sums under the row's offset h_i, so the splits add directly).  A row whose S^B leaves
// [2^-60, 2^60] -- the rows whose normalisers row_finish recomputes -- is evaluated again in
// FP64 under its exact largest exponent.
// pair(j) = P(x_i, y_j); sq: squared Euclidean (the norms enter the cost).
template <typename Pair>
__device__ __forceinline__ void dt_rows_finish_body(const Ctrl* ctrl, const Sched* sched, Consts kc, bool sq,
                                                    const double* __restrict__ xn2, const double* __restrict__ yn2,
                                                    const double2* __restrict__ gtab2, const double* __restrict__ r,
                                                    const double2* __restrict__ part,
                                                    const double* __restrict__ tpart, int P, int64_t i,
                                                    double* __restrict__ out, Pair&& pair) {
    double SB = 0.0, T = 0.0;
#pragma unroll 8   // independent loads in flight; the sum order is unchanged
    for (int p = 0; p < P; ++p) {
        SB += part[(int64_t)p * kc.n + i].y;
        T += tpart[(int64_t)p * kc.n + i];
    }
    if (SB >= 0x1p-60 && SB <= 0x1p+60) {
        out[i] = kc.s * r[i] * (T / SB);
        return;
    }
    const int64_t t = ctrl->t;
    const Sched sc = sched[t - ctrl->t_base];
    const double cB = 2.0 * kc.s * sc.lamB * LOG2E;
    const double2* __restrict__ g = gtab2 + (t & 1) * kc.m;
    double emax = -__builtin_inf();
    for (int64_t j = 0; j < kc.m; ++j) emax = fmax(emax, fma(cB, pair(j), g[j].y));
    const double xa = sq ? xn2[i] : 0.0;
    double S = 0.0, Tx = 0.0;
    for (int64_t j = 0; j < kc.m; ++j) {
        const double dot = pair(j);
        const double q = exp2(fma(cB, dot, g[j].y) - emax);
        S += q;
        Tx += q * fma(-2.0, dot, sq ? xa + yn2[j] : xa);
    }
    out[i] = kc.s * r[i] * (Tx / S);
}

template <int M, int D>
__global__ void dt_rows_finish(const Ctrl* ctrl, const Sched* sched, Consts kc, const double* __restrict__ xc,
                               const double* __restrict__ yc, const double* __restrict__ xn2,
                               const double* __restrict__ yn2, const double2* __restrict__ gtab2,
                               const double* __restrict__ r, const double2* __restrict__ part,
                               const double* __restrict__ tpart, int P, double* __restrict__ out) {
    if (halted(ctrl)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double x[D];
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = xc[i * D + k];
    dt_rows_finish_body(ctrl, sched, kc, M == METRIC_SQEUCLID, xn2, yn2, gtab2, r, part, tpart, P, i, out,
                        [&](int64_t j) { return pair_term<M, D>(x, yc + j * D, 0.0); });
}

// The same with the metric and the dimension at run time (the FP64 matrix-core sweeps).
__global__ void dt_rows_finish_dyn(const Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                                   const double* __restrict__ xc, const double* __restrict__ yc,
                                   const double* __restrict__ xn2, const double* __restrict__ yn2,
                                   const double2* __restrict__ gtab2, const double* __restrict__ r,
                                   const double2* __restrict__ part, const double* __restrict__ tpart, int P,
                                   double* __restrict__ out) {
    if (halted(ctrl)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    const double* __restrict__ xi = xc + i * D;
    dt_rows_finish_body(ctrl, sched, kc, kc.metric == METRIC_SQEUCLID, xn2, yn2, gtab2, r, part, tpart, P, i, out,
                        [&](int64_t j) { return pair_term_dyn(kc, D, xi, yc + j * D, 0.0); });
}

// ctrl->dt_cost = sum_i out_i, one block, fixed order (deterministic).
__global__ __launch_bounds__(1024) void dt_cost_total(Ctrl* ctrl, const double* __restrict__ vals, int64_t n) {
    if (halted(ctrl)) return;
    __shared__ double sh[1024];
    double a = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) a += vals[i];
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) ctrl->dt_cost = sh[0];
}

// ---------------------------------------------------------------------------
// Dual update (S5-S6 of Algorithm 2), residual, next column table, stop flag.
// State is double-buffered by iteration parity: iteration t reads buffer t&1 and
// writes buffer (t+1)&1, so the iterate that met the tolerance is never
// overwritten.
// ---------------------------------------------------------------------------
// Dual part of the D_t summand for one column, from the natural parameters of the mirror
// steps (thetabar = tanh abar, thetahat = tanh ahat, theta^t = tanh a):
//   D(thetabar||thetahat) - D(thetabar||theta^t)  per coordinate of def:DHa_explicit, with
//   (1 + tanh x)/2 = sigma(2x), is  2 sigma(2 abar) (a - ahat) + softplus(2 ahat) - softplus(2 a):
// exact where tanh rounds to +-1 (a step with c^alpha_j ~ alpha/m and |col_j - c_j| >> c^alpha_j).
__device__ __forceinline__ double softplus(double z) { return fmax(z, 0.0) + log1p(exp(-fabs(z))); }

__device__ __forceinline__ double dual_dt_term(double abar, double ahat, double a) {
    const double sig = 0.5 * (1.0 + tanh(abar));   // sigma(2 abar)
    return 2.0 * sig * (a - ahat) + softplus(2.0 * ahat) - softplus(2.0 * a);
}

struct DualBufs {
    double* nu[2];
    double* theta[2];
};

struct TraceCols {
    double *col_a, *col_b, *theta_bar, *theta_hat;
};

// The sums of a and (if asked for) b over the block (up to BLOCK threads, whole waves), valid in thread 0.
__device__ __forceinline__ double2 block_sums(double a, double b, bool both) {
    __shared__ double2 sh[BLOCK / 64];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        if (both) b += __shfl_xor(b, o, 64);
    }
    if (blockDim.x > 64) {
        __syncthreads();   // an earlier call's sums are read
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_double2(a, b);
        __syncthreads();
        a = b = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            a += sh[w].x;
            b += sh[w].y;
        }
    }
    return make_double2(a, b);
}

__device__ __forceinline__ void dual_update_body(Ctrl* ctrl, const Sched* sched, Consts kc,
                                                     const double2* __restrict__ cpart, int P,
                                                     const double* __restrict__ c,
                                                     const double* __restrict__ yn2, DualBufs buf,
                                                     double2* __restrict__ gtab2,
                                                     float2* __restrict__ gtabf, int64_t m_pad,
                                                     double* __restrict__ respart, TraceCols tr,
                                                     double* __restrict__ dtpart, int64_t bx_) {
    const bool first = bx_ == 0 && threadIdx.x == 0;
    if (first) ctrl->done_seen = ctrl->done;
    if (halted(ctrl)) return;
    const int64_t t = ctrl->t;
    if (first) {
        ctrl->t_row = t + 1;   // the next row sweep; this iteration is complete with complete_iteration
        ctrl->fallbacks += ctrl->fallbacks_row;
        ctrl->fallbacks_row = 0;
    }
    const Sched sc = sched[t - ctrl->t_base];
    const int64_t j = (int64_t)bx_ * blockDim.x + threadIdx.x;
    double res = 0.0, dtj = 0.0;
    int bad = 0;
    if (j < kc.m) {
        const double2 col = merge_splits(cpart, P, kc.m, j);
        const double colA = col.x, colB = col.y;
        const double* nu_r = buf.nu[t & 1];
        const double* th_r = buf.theta[t & 1];
        double* nu_w = buf.nu[(t + 1) & 1];
        double* th_w = buf.theta[(t + 1) & 1];
        const double cj = c[j];
        const double calpha = cj + kc.alpha_m;       // c^alpha = c + (alpha/m) 1
        const double nu = nu_r[j], th = th_r[j];
        const double a = atanh(th);
        // closed form of the dual mirror map (def:closed_form_opt)
        const double abar = a + kc.kappa * (colA - cj) / calpha;
        const double ahat = a + kc.kappa * (colB - cj) / calpha;
        const double tbar = tanh(abar);
        const double that = tanh(ahat);
        const double nun = nu + sc.w * (tbar - nu);            // step:lamp_main_nu
        const double thn = fmin(fmax(that, -kc.clipb), kc.clipb);  // tclip
        nu_w[j] = nun;
        th_w[j] = thn;
        // column table of iteration t+1
        const double nbn = nun + sc.w2 * (thn - nun);          // step:lamp_mid_nu at t+1
        const double base = kc.s * yn2[j];
        double2 gn;
        gn.x = -sc.lamB * LOG2E * (base + kc.K * nun);
        gn.y = -sc.lamC * LOG2E * (base + kc.K * nbn);
        gtab2[((t + 1) & 1) * kc.m + j] = gn;
        if (gtabf) gtabf[((t + 1) & 1) * m_pad + j] = make_float2((float)gn.x, (float)gn.y);
        res = fabs(colA - cj);
        bad = !(isfinite(nun) && isfinite(thn) && isfinite(colA) && isfinite(colB)) || fabs(th) >= 1.0;
        if (dtpart) {
            // D_t summand of this column (Lemma kl_diff, def:DHa_explicit):
            // c^a (D(tbar||that) - D(tbar||th)) + K colB (lam_{t+1} nu^{t+1} - lam_t nu^t)
            dtj = calpha * dual_dt_term(abar, ahat, a) + kc.K * colB * (sc.lamB * nun - sc.lamA * nu);
        }
        if (tr.col_a) tr.col_a[j] = colA;
        if (tr.col_b) tr.col_b[j] = colB;
        if (tr.theta_bar) tr.theta_bar[j] = tbar;
        if (tr.theta_hat) tr.theta_hat[j] = that;
    }
    // block reduction of the residual (and D_t summand; fixed order: deterministic)
    const double2 tot = block_sums(res, dtj, dtpart != nullptr);
    if (threadIdx.x == 0) {
        respart[bx_] = tot.x;
        if (dtpart) dtpart[bx_] = tot.y;
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(&ctrl->err, 1);
}

// Completes iteration t after its dual update (t_row = t + 1: a kernel boundary later, so that the
// block partials are visible; the dual update needs no device-scope fence and no last-block
// counter, which on a chip whose XCDs keep separate L2 caches write back the L2).  One block: the
// residual ||col(X^t) - c||_1 as a fixed-order sum over the block partials, the stop decision
// (iterates t >= 1 only; t = 0 is the product coupling of eta_0 = infinity), and otherwise the D_t
// summand of the step and t + 1.
template <int THREADS>
__device__ __forceinline__ void complete_iteration(Ctrl* ctrl, const Sched* sched, const double* __restrict__ respart,
                                                   const double* __restrict__ dtpart, int64_t nb) {
    const int64_t t = ctrl->t;   // the same control block for every thread: uniform
    if (ctrl->done != 0 || ctrl->t_row != t + 1) return;
    // BLOCK strided sums in BLOCK / 64 groups of 64 lanes, whatever the block: res_t, and with it the stop,
    // does not depend on which launch completes the iteration.  16 loads in flight a thread (one at a time,
    // the wave of row_finish took 32 turns of a full wait for the 2048 partials of 131072 columns).
    constexpr int R = BLOCK / THREADS, U = 16 / R;
    double a[R] = {}, b[R] = {};
    auto add = [&](const double* __restrict__ v, double (&sum)[R]) {
        if (nb <= 64) {
            if (threadIdx.x < nb) sum[0] = v[threadIdx.x];
            return;
        }
        for (int64_t k = threadIdx.x; k < nb; k += BLOCK * U) {
            double x[U][R];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int64_t q = k + u * BLOCK + r * THREADS;
                    x[u][r] = q < nb ? v[q] : 0.0;
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) sum[r] += x[u][r];
        }
    };
    add(respart, a);
    if (dtpart) add(dtpart, b);
    double2 sums = make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * THREADS >= nb) break;   // groups without a partial add 0
        const double2 g = block_sums(a[r], b[r], dtpart != nullptr);
        sums.x += g.x;
        sums.y += g.y;
    }
    __syncthreads();   // every thread has read t and done
    if (threadIdx.x != 0) return;
    const double tot = sums.x;
    ctrl->res_last = tot;
    if (ctrl->err) {
        ctrl->done = 1;
        ctrl->t_done = t;
    } else if (ctrl->tol > 0.0 && t >= 1 && tot <= ctrl->tol) {
        ctrl->done = 1;
        ctrl->t_done = t;
    } else {
        if (dtpart) {
            // the step is taken: its D_t summand joins the sum
            const Sched sc = sched[t - ctrl->t_base];
            ctrl->dt_acc += (sc.lamB - sc.lamA) * ctrl->dt_cost + sums.y;
        }
        ctrl->t = t + 1;
    }
}

// With nb > 0 the launch has one block more than the rows take, which completes the previous
// iteration (complete_iteration) while the rows' blocks merge this one's sums: the residual is
// looked at one row pass late, and a kernel per iteration is saved (4.5 us of 43 at 4096 x 4096).
// The rows' blocks go by done_seen, which no block of this launch writes.
__global__ void row_finish(Ctrl* ctrl, const Sched* sched, Consts kc, int D,
                           const double* __restrict__ xc, const double* __restrict__ yc,
                           const double2* __restrict__ gtab2, const double* __restrict__ r,
                           const double* __restrict__ xn2, const double2* __restrict__ part, int P,
                           double* __restrict__ H, RowVar* __restrict__ rowvar, double2* __restrict__ rowck,
                           double* __restrict__ log_za, double* __restrict__ log_zb, RowVarF32 rf,
                           const double* __restrict__ respart, int64_t nb) {
    if (nb > 0 && blockIdx.x == gridDim.x - 1) {
        complete_iteration<64>(ctrl, sched, respart, nullptr, nb);
        return;
    }
    row_finish_body(ctrl, sched, kc, D, xc, yc, gtab2, r, xn2, part, P, H, rowvar, rowck, log_za, log_zb, rf,
                    ctrl->done_seen, (int64_t)blockIdx.x);
}

__global__ __launch_bounds__(BLOCK) void dual_finish(Ctrl* ctrl, const Sched* sched, const double* __restrict__ respart,
                                                     const double* __restrict__ dtpart, int64_t nb) {
    complete_iteration<BLOCK>(ctrl, sched, respart, dtpart, nb);
}

__global__ __launch_bounds__(BLOCK) void dual_update(Ctrl* ctrl, const Sched* sched, Consts kc,
                                                     const double2* __restrict__ cpart, int P,
                                                     const double* __restrict__ c,
                                                     const double* __restrict__ yn2, DualBufs buf,
                                                     double2* __restrict__ gtab2,
                                                     float2* __restrict__ gtabf, int64_t m_pad,
                                                     double* __restrict__ respart, TraceCols tr,
                                                     double* __restrict__ dtpart) {
    dual_update_body(ctrl, sched, kc, cpart, P, c, yn2, buf, gtab2, gtabf, m_pad, respart, tr, dtpart, (int64_t)blockIdx.x);
}

// ---------------------------------------------------------------------------
// Deterministic single-block reductions.
// ---------------------------------------------------------------------------
// sums[q] = sum_i vals[q * stride + i], block q (each a fixed-order tree).
__global__ void reduce_sums(const double* __restrict__ vals, int64_t n, int64_t stride, double* __restrict__ out) {
    __shared__ double sh[1024];
    vals += blockIdx.x * stride;
    double acc = 0.0;
#pragma unroll 8   // independent loads in flight; the sum order is unchanged
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) acc += vals[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sh[0];
}

// Check of a marginal by one block of 1024 threads, into out[3]: the sum (fixed order), the first
// index whose entry is not a positive finite number (-1: none), that entry.  Eight loads in flight a
// thread.
__device__ __forceinline__ void marginal_stats_body(const double* __restrict__ a, int64_t len,
                                                    double* __restrict__ out) {
    __shared__ double sh[1024];
    __shared__ long long bad[1024];
    double acc = 0.0;
    long long first = -1;
    auto take = [&](double v, int64_t i) {
        acc += v;
        if (first < 0 && !(v > 0.0 && v <= 1.7976931348623157e308)) first = (long long)i;
    };
    int64_t i = threadIdx.x;
    const int64_t step = blockDim.x;
    for (; i + 7 * step < len; i += 8 * step) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = a[i + u * step];
#pragma unroll
        for (int u = 0; u < 8; ++u) take(v[u], i + u * step);
    }
    for (; i < len; i += step) take(a[i], i);
    sh[threadIdx.x] = acc;
    bad[threadIdx.x] = first;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sh[threadIdx.x] += sh[threadIdx.x + o];
            const long long b = bad[threadIdx.x + o];
            if (b >= 0 && (bad[threadIdx.x] < 0 || b < bad[threadIdx.x])) bad[threadIdx.x] = b;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = sh[0];
        out[1] = (double)bad[0];
        out[2] = bad[0] >= 0 ? a[bad[0]] : 0.0;
    }
}

// Both marginals of a call: block 0 checks r, block 1 c.
__global__ void marginal_stats(const double* __restrict__ r, int64_t n, const double* __restrict__ c, int64_t m,
                               double* __restrict__ out) {
    if (blockIdx.x == 0) marginal_stats_body(r, n, out);
    else marginal_stats_body(c, m, out + 3);
}

// ---------------------------------------------------------------------------
// The pair terms of the thread's own point against UNROLL streamed points (or one): coordinates
// in registers for a compile-time dimension (M, D); for the run-time metric and dimension
// (M = -1, D = 0) four coordinates at a time, each used for all UNROLL streamed points (one load
// of an own coordinate per 8 pairs; coordinate k of the point at src[k stride]).  The sum of a
// pair runs over k in order either way.  The pair term is symmetric in its points.
// ---------------------------------------------------------------------------
template <int M, int D>
struct OwnPoint {
    double x[D];
    __device__ __forceinline__ OwnPoint(const double* __restrict__ src, int64_t, int, const Consts&) {
#pragma unroll
        for (int k = 0; k < D; ++k) x[k] = src[k];
    }
    __device__ __forceinline__ double at(int k) const { return x[k]; }
    __device__ __forceinline__ double pair(const double* __restrict__ y) const { return pair_term<M, D>(x, y, 0.0); }
    __device__ __forceinline__ void pairs(const double* __restrict__ y, double (&out)[UNROLL]) const {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) out[u] = pair(y + u * D);
    }
};

template <>
struct OwnPoint<-1, 0> {
    const double* x;
    int64_t stride;
    int d;
    const Consts& kc;
    __device__ __forceinline__ OwnPoint(const double* __restrict__ src, int64_t stride_, int d_, const Consts& kc_)
        : x(src), stride(stride_), d(d_), kc(kc_) {}
    __device__ __forceinline__ double at(int k) const { return x[k * stride]; }
    __device__ __forceinline__ double pair(const double* __restrict__ y) const {
        if (kc.metric == METRIC_EXPLICIT) return pair_term_cost(kc, x[0], y[0], 0.0);
        double a = 0.0;
        for (int k = 0; k < d; ++k) a = accumulate(a, x[k * stride], y[k]);
        return kc.metric == METRIC_SQEUCLID ? a : fma(-0.5, a, 0.0);
    }
    __device__ __forceinline__ void pairs(const double* __restrict__ y, double (&out)[UNROLL]) const {
        if (kc.metric == METRIC_EXPLICIT) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) out[u] = pair_term_cost(kc, x[0], y[u], 0.0);
        } else if (kc.metric == METRIC_SQEUCLID) {
            run<METRIC_SQEUCLID>(y, out);
        } else if (kc.metric == METRIC_L1) {
            run<METRIC_L1>(y, out);
        } else {
            run<METRIC_LINF>(y, out);
        }
    }

private:
    template <int M>
    __device__ __forceinline__ static double add(double a, double u, double v) {
        if constexpr (M == METRIC_SQEUCLID) return fma(u, v, a);
        const double t = fabs(u - v);
        return M == METRIC_L1 ? a + t : fmax(a, t);
    }
    __device__ __forceinline__ double accumulate(double a, double u, double v) const {
        if (kc.metric == METRIC_SQEUCLID) return add<METRIC_SQEUCLID>(a, u, v);
        return kc.metric == METRIC_L1 ? add<METRIC_L1>(a, u, v) : add<METRIC_LINF>(a, u, v);
    }
    template <int M>
    __device__ __forceinline__ void run(const double* __restrict__ y, double (&out)[UNROLL]) const {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) out[u] = 0.0;
        int k = 0;
        for (; k + 4 <= d; k += 4) {
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = x[(k + q) * stride];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) out[u] = add<M>(out[u], v[q], y[u * d + k + q]);
        }
        for (; k < d; ++k) {
            const double v = x[k * stride];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) out[u] = add<M>(out[u], v, y[u * d + k]);
        }
        if constexpr (M != METRIC_SQEUCLID) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) out[u] = fma(-0.5, out[u], 0.0);
        }
    }
};

// term(P(own, y_j), j) for the UNROLL streamed points from j: their pair terms side by side, or, with more than
// 16 coordinates in registers, one or two at a time (a certificate by 1, 2, 4 and 8: 65536 x 65536 x 32 45.3, 52.3,
// 49.6, 49.4 ms, x 64 138, 123, 127, 127).
template <int M, int D, typename F>
__device__ __forceinline__ void terms(const OwnPoint<M, D>& own, const double* __restrict__ y, int Dm, int64_t j, F&& term) {
    if constexpr (D > 16) {
#pragma unroll(D <= 32 ? 1 : 2)
        for (int u = 0; u < UNROLL; ++u) term(own.pair(y + (j + u) * Dm), j + u);
    } else {
        double dot[UNROLL];
        own.pairs(y + j * Dm, dot);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) term(dot[u], j + u);
    }
}

// out[k len + i] = src[i d + k]: the own points' coordinates side by side for the run-time form.
__global__ void transpose_points(const double* __restrict__ src, int64_t len, int d, double* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < len * d) out[e] = src[(e % len) * d + e / len];
}

// Coordinates of the own points of a pass: point i, coordinate k at p[i point + k coord].
struct OwnPts {
    const double* p;
    int64_t point, coord;
};

// ---------------------------------------------------------------------------
// Certificate row sweep at the state's iterate (offsets from an A-only
// row_finish so that log2 p_ij = cfac (h_i + x~.y~) + g_j exactly):
//   vals[0][i] = r_i |sum_j p_ij - 1|                 (row infeasibility)
//   vals[1][i] = r_i sum_j C_ij p_ij                  (<C, X^t>)
//   vals[2][i] = r_i min_j (C_ij + K theta_j)         (D(theta), def:dual_spp)
//   vals[3][i] = r_i min_j (C_ij + K nu_j)            (D(nu))
//   psum_out[i] = sum_j p_ij                          (row sum of p, for Round)
// Terms as in the sweeps: FP64 exponent, FP32 exponential and sums over blocks of
// UNROLL columns, FP64 across blocks; the two minima in FP64.  Dm = run-time d.  Over XCD-aware
// column splits (sweep_block): part[p][i] = (sum_j p_ij, sum_j C_ij p_ij, the two minima) of
// split p, combined in order by cert_rows_merge.
// ---------------------------------------------------------------------------
// Groups of UNROLL streamed columns run with a compile-time count (their data are wave-uniform
// scalar loads issued together), and what depends on the column alone comes precomputed: 18
// vector slots a pair at d = 3, 4.5 -> 2.2 ms at 65536 x 65536.
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void cert_rows(Consts kc, int Dm, double cA, OwnPts xs,
                                                   const double* __restrict__ yc,
                                                   const double* __restrict__ xn2,
                                                   const double* __restrict__ yn2,
                                                   const double* __restrict__ gA,
                                                   const double* __restrict__ H,
                                                   const double* __restrict__ nu,
                                                   const double* __restrict__ theta,
                                                   double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j0 = sb.p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    const double h = H[i], xi2 = xn2[i];
    double psum = 0.0, csum = 0.0, mth = __builtin_inf(), mnu = __builtin_inf();
    float ap = 0.f, ac = 0.f;
    double K = kc.K;
    asm("" : "+v"(K));   // one scalar operand an instruction: the column's
    auto term = [&](double dot, int64_t j) {
        const float p = fexp2(fma_su(h + dot, cA, gA[j]));
        const double cij = kc.s * (xi2 + yn2[j] - 2.0 * dot);
        ap += p;
        ac = fmaf((float)cij, p, ac);
        mth = fmin(mth, fma(K, theta[j], cij));
        mnu = fmin(mnu, fma(K, nu[j], cij));
    };
    auto carry = [&] {
        psum += (double)ap;
        csum += (double)ac;
        ap = ac = 0.f;
    };
    int64_t j = j0;
    for (; j + UNROLL <= j1; j += UNROLL) {
        terms(own, yc, Dm, j, term);
        carry();
    }
    for (; j < j1; ++j) term(own.pair(yc + j * Dm), j);
    carry();
    double* o = part + (sb.p * kc.n + i) * 4;
    o[0] = psum;
    o[1] = csum;
    o[2] = mth;
    o[3] = mnu;
}

// The splits of the certificate row pass in order: the two sums added, the minima taken;
// mu (2 x n) keeps the minima for the entropic pass.
__global__ void cert_rows_merge(Consts kc, int P, const double* __restrict__ r, const double* __restrict__ part,
                                double* __restrict__ vals, double* __restrict__ psum_out, double* __restrict__ mu) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double psum = 0.0, csum = 0.0, mth = __builtin_inf(), mnu = __builtin_inf();
#pragma unroll 8
    for (int p = 0; p < P; ++p) {
        const double* o = part + ((int64_t)p * kc.n + i) * 4;
        psum += o[0];
        csum += o[1];
        mth = fmin(mth, o[2]);
        mnu = fmin(mnu, o[3]);
    }
    const double ri = r[i];
    vals[i] = ri * fabs(psum - 1.0);
    vals[kc.n + i] = ri * csum;
    vals[2 * kc.n + i] = ri * mth;
    vals[3 * kc.n + i] = ri * mnu;
    psum_out[i] = psum;
    mu[i] = mth;
    mu[kc.n + i] = mnu;
}

// ---------------------------------------------------------------------------
// Entropic dual values at eta = 1/lam > 0 (def:dual_spp_e): per row i and dual v in {theta, nu},
//   softmin_i(v) = mu_i - eta ln sum_j exp(-(C_ij + K v_j - mu_i) / eta),  mu_i = min_j (C_ij + K v_j),
// with the minimum exact in FP64 (from the certificate row pass), the terms (each <= 1, one of
// them 1) FP32 exponentials of FP64 arguments summed in FP32 over blocks of UNROLL columns and in
// FP64 across them and across the splits (in order).
//   part[p][i] = (split p's sum for theta, for nu);  vals[0][i] = r_i softmin_i(theta), vals[1][i] likewise.
// ---------------------------------------------------------------------------
// The exponent is f ((C_ij + K v_j) - mu_i), f = -lam LOG2E, the parenthesis formed with the operations that gave
// mu_i: it is exactly 0 at the minimum and not positive elsewhere, so that a row's sum lies in [1, m] for every lam.
// Where the parts are small enough it is (2 s lam LOG2E P_ij + b_j) + (f s |x~_i|^2 - f mu_i) instead, with
// b_j = f (s |y~_j|^2 + K v_j) per column from cert_soft_cols: 15 vector slots a pair at d = 3 instead of 20, 1.9
// instead of 2.4 ms at 65536 x 65536.  What f times the parts' rounding leaves over moves an exponent by
// 2^-52 of their sum: with parts up to SOFT_PARTS by 2^-16, and a dual value, 1 / lam times that, by less than its own
// rounding; 2^22 further on the sums would run out of the FP32 exponents.  (2 s lam LOG2E P_ij is no larger than the
// other parts together, or the exponent is as large as it.)  Per wave, by its rows' parts and the largest of a column.
constexpr double SOFT_PARTS = 0x1p36;

__global__ void cert_soft_cols(Consts kc, double lam, const double* __restrict__ yn2,
                               const double* __restrict__ nu, const double* __restrict__ theta,
                               double2* __restrict__ out, unsigned long long* __restrict__ largest) {
    const double f = -lam * LOG2E;
    double most = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < kc.m; j += (int64_t)gridDim.x * blockDim.x) {
        const double b = kc.s * yn2[j], kt = kc.K * theta[j], kn = kc.K * nu[j];
        out[j] = make_double2(f * (b + kt), f * (b + kn));
        most = fmax(most, -f * (b + fmax(fabs(kt), fabs(kn))));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) most = fmax(most, __shfl_xor(most, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(largest, (unsigned long long)__double_as_longlong(most));
}

template <int M, int D>
__global__ __launch_bounds__(BLOCK) void cert_soft_rows(Consts kc, int Dm, double lam, OwnPts xs,
                                                        const double* __restrict__ yc,
                                                        const double* __restrict__ xn2,
                                                        const double* __restrict__ yn2,
                                                        const double* __restrict__ nu,
                                                        const double* __restrict__ theta,
                                                        const double2* __restrict__ cols,
                                                        const double* __restrict__ largest,
                                                        const double* __restrict__ mu,
                                                        double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j0 = sb.p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    const double f = -lam * LOG2E, xi2 = xn2[i], mth = mu[i], mnu = mu[kc.n + i];
    double sth = 0.0, snu = 0.0;
    float at = 0.f, an = 0.f;
    auto carry = [&] {
        sth += (double)at;
        snu += (double)an;
        at = an = 0.f;
    };
    auto run = [&](auto&& term) {
        int64_t j = j0;
        for (; j + UNROLL <= j1; j += UNROLL) {
            terms(own, yc, Dm, j, term);
            carry();
        }
        for (; j < j1; ++j) term(own.pair(yc + j * Dm), j);
        carry();
    };
    const double parts = *largest - f * (kc.s * xi2 + fmax(fabs(mth), fabs(mnu)));
    if (!__all(parts <= SOFT_PARTS)) {
        double K = kc.K;
        asm("" : "+v"(K));   // one scalar operand an instruction: the column's
        run([&](double dot, int64_t j) {
            const double cij = kc.s * (xi2 + yn2[j] - 2.0 * dot);
            at += fexp2(f * (fma(K, theta[j], cij) - mth));
            an += fexp2(f * (fma(K, nu[j], cij) - mnu));
        });
    } else {
        const double c = -2.0 * f * kc.s, rth = f * (kc.s * xi2 - mth), rnu = f * (kc.s * xi2 - mnu);
        run([&](double dot, int64_t j) {
            const double2 b = cols[j];
            at += fexp2(fma_su(dot, c, b.x) + rth);
            an += fexp2(fma_su(dot, c, b.y) + rnu);
        });
    }
    double* o = part + (sb.p * kc.n + i) * 2;
    o[0] = sth;
    o[1] = snu;
}

__global__ void cert_soft_merge(Consts kc, int P, double lam, const double* __restrict__ r,
                                const double* __restrict__ mu, const double* __restrict__ part,
                                double* __restrict__ vals) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double sth = 0.0, snu = 0.0;
#pragma unroll 8
    for (int p = 0; p < P; ++p) {
        sth += part[((int64_t)p * kc.n + i) * 2];
        snu += part[((int64_t)p * kc.n + i) * 2 + 1];
    }
    const double ri = r[i];
    vals[i] = ri * (mu[i] - log(sth) / lam);
    vals[kc.n + i] = ri * (mu[kc.n + i] - log(snu) / lam);
}

// ---------------------------------------------------------------------------
// Round (Algorithm 3) of the same X = diag(r) p on the device, without forming it:
//   step 1  xr_i = min(r_i / row_i(X), 1) = min(1 / sum_j p_ij, 1)
//   step 2  X' = diag(xr) X;  y_j = min(c_j / col_j(X'), 1);  X'' = X' diag(y)
//   step 3  dr = r - row(X''),  dc = c - col(X'') = c - y * col(X')
//   step 4  Round(X) = X'' + dr dc^T / ||dr||_1
// so that <C, Round(X)> = <C, X''> + dr^T C dc / ||dr||_1, where for the squared
// Euclidean cost on centred points
//   (C dc)_i = s (||x~_i||^2 sum_j dc_j + sum_j dc_j ||y~_j||^2 - 2 x~_i . sum_j dc_j y~_j)
// is O(d) per row once the column sums are known.  The pair passes use the terms of
// the certificate row sweep (FP32 exponentials, FP64 sums), the O(n + m) steps FP64.
// ---------------------------------------------------------------------------
// w_i = xr_i r_i rounded to FP32 (the weight of the pair terms).
__global__ void round_row_factors(Consts kc, const double* __restrict__ psum, const double* __restrict__ r,
                                  double* __restrict__ xr, float* __restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    const double x = fmin(1.0 / psum[i], 1.0);
    xr[i] = x;
    w[i] = (float)(x * r[i]);
}

// part[p][j] = sum over the rows i of split p of xr_i r_i p_ij (one thread per
// column, rows in order); round_cols_merge adds the splits in order: colp_j.
// 9 vector slots a pair at d = 3 (the weights were multiplied and rounded per pair before: 3.4 ->
// 1.2 ms at 65536 x 65536).
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void round_cols(Consts kc, int Dm, double cA, const double* __restrict__ xc,
                                                    OwnPts ys, const double* __restrict__ gA,
                                                    const double* __restrict__ H, const float* __restrict__ w,
                                                    double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.n, split);
    const int64_t j = sb.bx * BLOCK + threadIdx.x;
    if (j >= kc.m) return;
    const int64_t p = sb.p;
    const int64_t i0 = p * split;
    const int64_t i1 = min(kc.n, i0 + split);
    const OwnPoint<M, D> own(ys.p + j * ys.point, ys.coord, Dm, kc);
    const double g = gA[j];
    double acc = 0.0;
    float a = 0.f;
    auto term = [&](double dot, int64_t i) { a = fmaf(w[i], fexp2(fma(cA, H[i] + dot, g)), a); };
    auto carry = [&] {
        acc += (double)a;
        a = 0.f;
    };
    int64_t i = i0;
    for (; i + UNROLL <= i1; i += UNROLL) {
        terms(own, xc, Dm, i, term);
        carry();
    }
    for (; i < i1; ++i) term(own.pair(xc + i * Dm), i);
    carry();
    part[p * kc.m + j] = acc;
}

__global__ void round_cols_merge(Consts kc, const double* __restrict__ part, int P, double* __restrict__ colp) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= kc.m) return;
    double a = part[j];
    for (int p = 1; p < P; ++p) a += part[(int64_t)p * kc.m + j];
    colp[j] = a;
}

// y_j = min(c_j / colp_j, 1), dc_j = c_j - y_j colp_j, and (y_j, 1 - y_j) in FP32 for the pair terms.
__global__ void round_col_factors(Consts kc, const double* __restrict__ c, const double* __restrict__ colp,
                                  double* __restrict__ y, double* __restrict__ dc, float2* __restrict__ yf) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= kc.m) return;
    const double yj = colp[j] > 0.0 ? fmin(c[j] / colp[j], 1.0) : 1.0;
    y[j] = yj;
    dc[j] = c[j] - yj * colp[j];
    yf[j] = make_float2((float)yj, (float)(1.0 - yj));
}

// Rows of X'': dr_i = r_i - xr_i r_i sum_j p_ij y_j and cpp_i = xr_i r_i sum_j C_ij p_ij y_j.
// dr is formed as r_i (1 - xr_i psum_i) + xr_i r_i sum_j p_ij (1 - y_j) (the same value)
// with psum_i recomputed in this pass: no difference of two nearly equal sums.  Over XCD-aware
// column splits: part[p][i] = split p's three sums, combined in order by round_rows_merge.
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void round_rows(Consts kc, int Dm, double cA, OwnPts xs,
                                                    const double* __restrict__ yc, const double* __restrict__ xn2,
                                                    const double* __restrict__ yn2, const double* __restrict__ gA,
                                                    const double* __restrict__ H, const float2* __restrict__ yf,
                                                    double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j0 = sb.p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    const double h = H[i], xi2 = xn2[i];
    double ps = 0.0, pq = 0.0, cs = 0.0;
    float a = 0.f, b = 0.f, e = 0.f;
    auto term = [&](double dot, int64_t j) {
        const float p = fexp2(fma_su(h + dot, cA, gA[j]));
        const float2 y = yf[j];
        const float py = p * y.x;
        a += p;
        b = fmaf(p, y.y, b);
        e = fmaf((float)(kc.s * (xi2 + yn2[j] - 2.0 * dot)), py, e);
    };
    auto carry = [&] {
        ps += (double)a;
        pq += (double)b;
        cs += (double)e;
        a = b = e = 0.f;
    };
    int64_t j = j0;
    for (; j + UNROLL <= j1; j += UNROLL) {
        terms(own, yc, Dm, j, term);
        carry();
    }
    for (; j < j1; ++j) term(own.pair(yc + j * Dm), j);
    carry();
    double* o = part + (sb.p * kc.n + i) * 3;
    o[0] = ps;
    o[1] = pq;
    o[2] = cs;
}

__global__ void round_rows_merge(Consts kc, int P, const double* __restrict__ r, const double* __restrict__ xr,
                                 const double* __restrict__ part, double* __restrict__ dr, double* __restrict__ cpp) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double ps = 0.0, pq = 0.0, cs = 0.0;
#pragma unroll 8
    for (int p = 0; p < P; ++p) {
        const double* o = part + ((int64_t)p * kc.n + i) * 3;
        ps += o[0];
        pq += o[1];
        cs += o[2];
    }
    const double w = xr[i] * r[i];
    dr[i] = r[i] * (1.0 - xr[i] * ps) + w * pq;
    cpp[i] = w * cs;
}

// Column sums of dc: S[k] = sum_j dc_j y~_jk (k < D), S[D] = sum_j dc_j,
// S[D+1] = sum_j dc_j ||y~_j||^2; block b computes S[b] in a fixed order.
__global__ void round_col_sums(Consts kc, int D, const double* __restrict__ yc, const double* __restrict__ yn2,
                               const double* __restrict__ dc, double* __restrict__ S) {
    __shared__ double sh[BLOCK];
    const int b = blockIdx.x;
    double acc = 0.0;
    for (int64_t j = threadIdx.x; j < kc.m; j += BLOCK) {
        const double v = b < D ? yc[j * D + b] : (b == D ? 1.0 : yn2[j]);
        acc = fma(dc[j], v, acc);
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = BLOCK / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) S[b] = sh[0];
}

// (C dc)_i by a pass over all pairs (the l1 / l_inf costs, whose C dc has no closed form;
// C_ij = -2 s P(x~_i, y~_j)): part[p][i] = sum of P(x~_i, y~_j) dc_j over column split p, FP64.  One
// thread a row and a run-time dimension took 14.2 ms for 13378 x 38523 x 3, l1, against 0.3 ms of the
// other pair passes; split and compiled like them 0.13 ms.
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void round_rank_one_pairs(Consts kc, int Dm, OwnPts xs,
                                                              const double* __restrict__ yc,
                                                              const double* __restrict__ dc,
                                                              double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j1 = min(kc.m, (sb.p + 1) * split);
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    double acc = 0.0;
    int64_t j = sb.p * split;
    for (; j + UNROLL <= j1; j += UNROLL) {
        double dot[UNROLL];
        own.pairs(yc + j * Dm, dot);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) acc = fma(dot[u], dc[j + u], acc);
    }
    for (; j < j1; ++j) acc = fma(own.pair(yc + j * Dm), dc[j], acc);
    part[sb.p * kc.n + i] = acc;
}

// t_i = dr_i (C dc)_i and |dr_i| from the splits' sums, in split order.
__global__ void round_rank_one_merge(Consts kc, int P, const double* __restrict__ dr, const double* __restrict__ part,
                                     double* __restrict__ t, double* __restrict__ absdr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double acc = 0.0;
#pragma unroll 8
    for (int p = 0; p < P; ++p) acc += part[(int64_t)p * kc.n + i];
    t[i] = dr[i] * (-2.0 * kc.s * acc);
    absdr[i] = fabs(dr[i]);
}

// t_i = dr_i (C dc)_i and |dr_i|.
__global__ void round_rank_one(Consts kc, int D, const double* __restrict__ xc, const double* __restrict__ xn2,
                               const double* __restrict__ dr, const double* __restrict__ S,
                               double* __restrict__ t, double* __restrict__ absdr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    double xs = 0.0;
    for (int k = 0; k < D; ++k) xs = fma(xc[i * D + k], S[k], xs);
    t[i] = dr[i] * kc.s * (xn2[i] * S[D] + S[D + 1] - 2.0 * xs);
    absdr[i] = fabs(dr[i]);
}

// c_j * theta_j products for <c, theta>, <c, nu>; clears a word for a later maximum.
__global__ void col_products(Consts kc, const double* __restrict__ c, const double* __restrict__ a,
                             const double* __restrict__ b, double* __restrict__ out,
                             unsigned long long* __restrict__ clear) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j == 0) *clear = 0ull;
    if (j >= kc.m) return;
    out[j] = c[j] * a[j];
    out[kc.m + j] = c[j] * b[j];
}

// ---------------------------------------------------------------------------
// Adjoint sweep (envelope gradient), one pass over the pairs: per row i and column split p,
// with unnormalised weights q_ij = 2^(cfac P_ij + g_j - M_ip) (g_j = g^A_j of X^t), the
// partial sums Z_ip = sum_j q_ij and S1_ip (d values) and the split's offset M_ip, an
// integer that each lane raises to ceil(max e) whenever a block of columns exceeds it
// (the first block sets it), so every term is at most 1 and a raise rescales the sums
// exactly by a power of two.  grad_i = 2 s r_i (c_x Z_i x~_i - S1_i) / Z_i, the
// normaliser cancelling in the ratio:
//   squared Euclidean (dC/dx = 2 s (x - y)):  c_x = 1, S1 = sum_j q_ij y~_j;
//   l1 (dC/dx_k = s sign(x_k - y_k)):       c_x = 0, S1_k = -1/2 sum_j q_ij sign(x_k - y_jk);
//   l_inf (the coordinate k* of the largest |x_k - y_k|, the first one on ties):
//                                           c_x = 0, S1_k = -1/2 sum_j q_ij sign(x_k - y_jk) [k = k*].
// (sign(0) = 0: the subgradient at a kink.)  part: [P][n][D+2] = (M, Z, S1).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float sgnf(double v) { return v > 0.0 ? 1.f : (v < 0.0 ? -1.f : 0.f); }

// The one-pass row sweeps at X^t -- the adjoint above and the transport cost
// <C, X^t> = sum_i r_i sum_j p_ij C_ij -- share the exponent assembly and the offset
// handling; what each adds per column is a policy:
//   Col     the column record, read with a few wide scalar loads;
//   W       the number of sums (FP32 within a block of columns, FP64 across blocks);
//   block   called with the dot products' initial value hb of each block of columns;
//   add     accumulates one column with weight q, given ph = hb + P_ij.

// One column's data for the adjoint: y~_j in FP64 (dot product), g^A_j, y~_j in FP32 (S1).
template <int D>
struct alignas(16) AdjCol {
    double y[D];
    double g;
    float yf[D];
};

// The adjoint's sums: Z and S1 (d values, in the form of the metric).
template <int M, int D>
struct GradSums {
    using Col = AdjCol<D>;
    static constexpr int W = D + 1;
    __device__ __forceinline__ void block(double) {}
    __device__ __forceinline__ void add(const double (&x)[D], const Col& c, double, float q, float (&a)[W]) const {
        a[0] += q;
        if constexpr (M == METRIC_SQEUCLID) {
#pragma unroll
            for (int k = 0; k < D; ++k) a[1 + k] = fmaf(q, c.yf[k], a[1 + k]);
        } else if constexpr (M == METRIC_L1) {
#pragma unroll
            for (int k = 0; k < D; ++k) a[1 + k] = fmaf(-0.5f * q, sgnf(x[k] - c.y[k]), a[1 + k]);
        } else {
            int ks = 0;
            double best = -1.0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const double t = fabs(x[k] - c.y[k]);
                if (t > best) {
                    best = t;
                    ks = k;
                }
            }
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (k == ks) a[1 + k] = fmaf(-0.5f * q, sgnf(x[k] - c.y[k]), a[1 + k]);
        }
    }
};

// One column's data for the transport cost: y~_j (FP64), g^A_j, |y~_j|^2.
template <int D>
struct alignas(16) CostCol {
    double y[D];
    double g;
    double yn2;
};

// The transport cost's sums: Z and S_C = sum_j q_ij C_ij / s.  C_ij / s = |x~_i|^2 + |y~_j|^2
// - 2 P_ij is taken from the exponent's dot product ph = hb + P_ij as
// (|x~_i|^2 + 2 hb + |y~_j|^2) - 2 ph, two FP64 operations per pair (the norms are zero
// for l1 / l_inf, where P_ij = -dist / 2); each term is nonnegative, so the FP32 block sums
// lose no digits to cancellation.
template <int M, int D>
struct CostSums {
    using Col = CostCol<D>;
    static constexpr int W = 2;
    double xn2 = 0.0, a = 0.0;
    __device__ __forceinline__ void block(double hb) { a = xn2 + 2.0 * hb; }
    __device__ __forceinline__ void add(const double (&)[D], const Col& c, double ph, float q, float (&s)[W]) const {
        s[0] += q;
        const double cs = fma(-2.0, ph, M == METRIC_SQEUCLID ? a + c.yn2 : a);
        s[1] = fmaf(q, (float)cs, s[1]);
    }
};

// The row sums alone (Z): X^t's row normalisers in one pass, for the adjoint with respect to
// y, whose column pass weights each row by r_i / Z_i.
template <int D>
struct NormSums {
    using Col = CostCol<D>;
    static constexpr int W = 1;
    __device__ __forceinline__ void block(double) {}
    __device__ __forceinline__ void add(const double (&)[D], const Col&, double, float q, float (&s)[W]) const {
        s[0] += q;
    }
};

template <int D>
__global__ void adjoint_pack(int64_t m, const double* __restrict__ yc, const float* __restrict__ ycf,
                             const double* __restrict__ gA, AdjCol<D>* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    AdjCol<D> c;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        c.y[k] = yc[j * D + k];
        c.yf[k] = ycf[j * D + k];
    }
    c.g = gA[j];
    out[j] = c;
}

template <int D>
__global__ void cost_pack(int64_t m, const double* __restrict__ yc, const double* __restrict__ yn2,
                          const double* __restrict__ gA, CostCol<D>* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    CostCol<D> c;
#pragma unroll
    for (int k = 0; k < D; ++k) c.y[k] = yc[j * D + k];
    c.g = gA[j];
    c.yn2 = yn2[j];
    out[j] = c;
}

// Per row i and column split p: the split's offset M_ip, an integer that each lane raises to
// ceil(max e) whenever a block of columns exceeds it (the first block sets it), so every
// term is at most 1 and a raise rescales the sums exactly by a power of two; then the W sums
// of the policy.  part: [P][n][W + 1] = (M, sums); an empty split writes M = -inf.
template <int M, int D, class Pol>
__device__ __forceinline__ void weighted_row_sums(const Consts& kc, double cA, const double* __restrict__ xc,
                                                  const typename Pol::Col* __restrict__ cols, Pol pol,
                                                  double* __restrict__ part, int64_t split) {
    constexpr int W = Pol::W;
    using Col = typename Pol::Col;
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    const int64_t p = sb.p;
    const int64_t j0 = p * split;
    const int64_t j1 = min(kc.m, j0 + split);
    const int64_t ii = i < kc.n ? i : kc.n - 1;
    double x[D];
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = xc[ii * D + k];
    double off = 0.0;      // M: integer offset of this lane's exponents
    double h = 0.0;        // -M / cfac, the dot products' initial value
    bool first = true;
    double s[W];
#pragma unroll
    for (int w = 0; w < W; ++w) s[w] = 0.0;
    // raise the offset by ceil(bm) (bm: the largest exponent under the current offset),
    // rescaling the sums exactly; returns the raise
    auto raise = [&](double bm) {
        const double sh = ceil(bm);
#pragma unroll
        for (int w = 0; w < W; ++w) s[w] = ldexp(s[w], -(int)sh);
        off += sh;
        h = -off / cA;
        return sh;
    };
    // blocks of UNROLL columns with a compile-time trip count (the column data are
    // wave-uniform scalar loads, issued together); the offset is checked once per block
    const int64_t nfull = (j1 - j0) / UNROLL;
    const Col* __restrict__ cp = cols + j0;
    for (int64_t c = 0; c < nfull; ++c, cp += UNROLL) {
        const double hb = h;
        double ph[UNROLL], e[UNROLL];
        float ef[UNROLL];
        float bm = -__builtin_inff();
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            ph[u] = pair_term<M, D>(x, cp[u].y, hb);
            e[u] = fma_su(ph[u], cA, cp[u].g);
            ef[u] = (float)e[u];
            bm = fmaxf(bm, ef[u]);
        }
        if (first || bm > 0.f) {   // rare after the first block
            double bmd = e[0];
#pragma unroll
            for (int u = 1; u < UNROLL; ++u) bmd = fmax(bmd, e[u]);
            const double sh = raise(bmd);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) ef[u] = (float)(e[u] - sh);
            first = false;
        }
        pol.block(hb);
        float a[W];
#pragma unroll
        for (int w = 0; w < W; ++w) a[w] = 0.f;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) pol.add(x, cp[u], ph[u], __builtin_amdgcn_exp2f(ef[u]), a);
#pragma unroll
        for (int w = 0; w < W; ++w) s[w] += (double)a[w];
    }
    // the remaining columns one at a time
    for (int64_t j = j0 + nfull * UNROLL; j < j1; ++j) {
        const double hb = h;
        const double ph = pair_term<M, D>(x, cols[j].y, hb);
        double e = fma_su(ph, cA, cols[j].g);
        if (first || e > 0.0) {
            e -= raise(e);
            first = false;
        }
        pol.block(hb);
        float a[W];
#pragma unroll
        for (int w = 0; w < W; ++w) a[w] = 0.f;
        pol.add(x, cols[j], ph, fexp2(e), a);
#pragma unroll
        for (int w = 0; w < W; ++w) s[w] += (double)a[w];
    }
    if (i < kc.n) {
        double* o = part + (p * kc.n + i) * (W + 1);
        o[0] = first ? -__builtin_inf() : off;   // an empty split contributes nothing
#pragma unroll
        for (int w = 0; w < W; ++w) o[1 + w] = s[w];
    }
}

// part: [P][n][D + 2] = (M, Z, S1).
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void adjoint_sweep(Consts kc, double cA, const double* __restrict__ xc,
                                                       const AdjCol<D>* __restrict__ cols,
                                                       double* __restrict__ part, int64_t split) {
    weighted_row_sums<M, D>(kc, cA, xc, cols, GradSums<M, D>{}, part, split);
}

// part: [P][n][3] = (M, Z, S_C).
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void cost_sweep(Consts kc, double cA, const double* __restrict__ xc,
                                                    const double* __restrict__ xn2,
                                                    const CostCol<D>* __restrict__ cols,
                                                    double* __restrict__ part, int64_t split) {
    const int64_t i = sweep_block(kc.m, split).bx * BLOCK + threadIdx.x;
    CostSums<M, D> pol;
    if constexpr (M == METRIC_SQEUCLID) pol.xn2 = xn2[i < kc.n ? i : kc.n - 1];
    weighted_row_sums<M, D>(kc, cA, xc, cols, pol, part, split);
}

// part: [P][n][2] = (M, Z).
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void norm_sweep(Consts kc, double cA, const double* __restrict__ xc,
                                                    const CostCol<D>* __restrict__ cols,
                                                    double* __restrict__ part, int64_t split) {
    weighted_row_sums<M, D>(kc, cA, xc, cols, NormSums<D>{}, part, split);
}

// Split partials of a row under their own offsets (o[0] = M_p; -inf: no finite term) at the common
// offset: 2^(M_p - off) v, exact.
__device__ __forceinline__ double at_offset(double m, double v, double off) {
    return m > -__builtin_inf() ? ldexp(v, (int)(m - off)) : 0.0;
}

// The largest offset of row i's partials (W doubles each).
__device__ __forceinline__ double common_offset(const double* __restrict__ part, int P, int64_t n, int W, int64_t i) {
    double off = -__builtin_inf();
#pragma unroll 16
    for (int p = 0; p < P; ++p) off = fmax(off, part[((int64_t)p * n + i) * W]);
    return off;
}

// The merges run one wave a block, with 16 splits' loads in flight: they are bound by latency, and
// blocks of 256 rows left most of the chip idle (941 rows of 107 splits: 29 us on 4 CUs).
//
// X^t's row data for the column-side adjoint from the splits' (M, Z) at their common offset:
// sigma_i = M + log2 Z (base 2), k_i = -sigma_i / cfac, so that
// X_ij = r_i 2^(cfac (k_i + P_ij) + g_j); wA = wB = r_i.
__global__ __launch_bounds__(64) void norm_finish(Consts kc, int P, double cA, const double* __restrict__ r,
                            const double* __restrict__ part, RowVar* __restrict__ rowvar) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    const double off = common_offset(part, P, kc.n, 2, i);
    double z = 0.0;
#pragma unroll 16
    for (int p = 0; p < P; ++p) {
        const double* o = part + ((int64_t)p * kc.n + i) * 2;
        z += at_offset(o[0], o[1], off);
    }
    RowVar rv;
    rv.k = -(off + log2(z)) / cA;
    rv.wA = rv.wB = (float)r[i];
    rowvar[i] = rv;
}

// Rows' weighted sums for the dimensions without a packed form above: weights q_ij = 2^(e_ij - M) under
// the lane's running integer offset M, every sum FP64.  term(q, dot, j) takes the weights and pair terms
// of UNROLL streamed points from j (or one); rescale(sh) multiplies the sums by 2^sh (exact).
template <typename Own, typename Rescale, typename Term>
__device__ __forceinline__ double offset_weights(const Own& own, int Dm, double cA, const double* __restrict__ yc,
                                                 const double* __restrict__ gA, int64_t j0, int64_t j1,
                                                 Rescale&& rescale, Term&& term) {
    double off = -__builtin_inf();
    auto run = [&](auto cnt, int64_t j) {
        constexpr int U = decltype(cnt)::value;
        double dot[U], q[U], top = -__builtin_inf();
        if constexpr (U == 1) dot[0] = own.pair(yc + j * Dm);
        else own.pairs(yc + j * Dm, dot);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            q[u] = fma(cA, dot[u], gA[j + u]);
            top = fmax(top, q[u]);
        }
        if (top > off) {   // raise the offset to the next integer
            const double nm = ceil(top);
            if (off > -__builtin_inf()) rescale((int)(off - nm));
            off = nm;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) q[u] = (double)fexp2(q[u] - off);
        term(q, dot, j);
    };
    int64_t j = j0;
    for (; j + UNROLL <= j1; j += UNROLL) run(std::integral_constant<int, UNROLL>{}, j);
    for (; j < j1; ++j) run(std::integral_constant<int, 1>{}, j);
    return off;
}

// The transport cost.  part as above.
template <int M, int D>
__global__ __launch_bounds__(BLOCK) void cost_sweep_any(Consts kc, int Dm, double cA, OwnPts xs,
                                                        const double* __restrict__ yc,
                                                        const double* __restrict__ xn2,
                                                        const double* __restrict__ yn2,
                                                        const double* __restrict__ gA,
                                                        double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j0 = sb.p * split;
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    const double x2 = xn2[i];
    double s0 = 0.0, sc = 0.0;
    const double off = offset_weights(
        own, Dm, cA, yc, gA, j0, min(kc.m, j0 + split),
        [&](int sh) {
            s0 = ldexp(s0, sh);
            sc = ldexp(sc, sh);
        },
        [&](const auto& q, const auto& dot, int64_t j) {
            constexpr int U = sizeof(q) / sizeof(double);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s0 += q[u];
                sc += q[u] * fma(-2.0, dot[u], x2 + yn2[j + u]);
            }
        });
    double* o = part + (sb.p * kc.n + i) * 3;
    o[0] = off;
    o[1] = s0;
    o[2] = sc;
}

// Row i's share of the transport cost, s r_i S_C / Z, from the splits' (M, Z, S_C) brought to
// their common offset (exact powers of two).
__global__ __launch_bounds__(64) void cost_finish(Consts kc, int P, const double* __restrict__ r, const double* __restrict__ part,
                            double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kc.n) return;
    const double off = common_offset(part, P, kc.n, 3, i);
    double z = 0.0, c = 0.0;
#pragma unroll 16
    for (int p = 0; p < P; ++p) {
        const double* o = part + ((int64_t)p * kc.n + i) * 3;
        z += at_offset(o[0], o[1], off);
        c += at_offset(o[0], o[2], off);
    }
    out[i] = kc.s * r[i] * (c / z);
}

// Adds the derivatives of U streamed points from y in the coordinates c0 + k, k < nc <= KC, to s[k] with
// their weights w_u >= 0: w_u y_k for the squared Euclidean cost, w_u / 2 sgn(y_k - x_k) for l1, the
// same on the coordinate of the largest |x_k - y_k| (the first on ties) for l_inf; FP64.
template <int D, int KC, int U, typename Own>
__device__ __forceinline__ void add_derivatives(int metric, int Dm, int c0, int nc, const double (&w)[U],
                                                const Own& own, const double* __restrict__ y, double (&s)[KC]) {
    if (metric == METRIC_SQEUCLID) {
#pragma unroll
        for (int k = 0; k < KC; k += 4) {
            if constexpr (D == 0) __builtin_amdgcn_sched_barrier(0);   // one block's scalar loads in flight
            if (k + 4 <= nc) {                   // uniform
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int v = k; v < k + 4 && v < KC; ++v) s[v] = fma(w[u], y[u * Dm + c0 + v], s[v]);
            } else {
#pragma unroll
                for (int v = k; v < k + 4 && v < KC; ++v)
                    if (v < nc)
#pragma unroll
                        for (int u = 0; u < U; ++u) s[v] = fma(w[u], y[u * Dm + c0 + v], s[v]);
            }
        }
        return;
    }
    int ks[U];
    if (metric == METRIC_LINF) {
        double best[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ks[u] = 0;
            best[u] = -1.0;
        }
        auto scan = [&](int k) {
            const double xk = own.at(k);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double t = fabs(xk - y[u * Dm + k]);
                if (t > best[u]) {
                    best[u] = t;
                    ks[u] = k;
                }
            }
        };
        if constexpr (D > 0) {
#pragma unroll
            for (int k = 0; k < D; ++k) scan(k);
        } else {
            for (int k = 0; k < Dm; ++k) scan(k);
        }
    }
#pragma unroll
    for (int v = 0; v < KC; ++v) {
        if constexpr (D == 0) __builtin_amdgcn_sched_barrier(0);
        if (v >= nc) continue;   // uniform
        const double xk = own.at(c0 + v);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double t = y[u * Dm + c0 + v] - xk;
            const bool on = metric == METRIC_L1 || ks[u] == c0 + v;
            s[v] += on && t != 0.0 ? copysign(0.5 * w[u], t) : 0.0;
        }
    }
}

// The gradient sums for the dimensions without a packed form: KC of them a block (blockIdx.y the chunk),
// in registers.  The run-time form (M = -1, D = 0) recomputes the weights for every chunk of at most
// 32 coordinates.  part as adjoint_sweep's.
template <int M, int D, int KC>
__global__ __launch_bounds__(BLOCK) void adjoint_sweep_any(Consts kc, int Dm, int chunk, double cA, OwnPts xs,
                                                           const double* __restrict__ yc,
                                                           const double* __restrict__ gA,
                                                           double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.m, split);
    const int64_t i = sb.bx * BLOCK + threadIdx.x;
    if (i >= kc.n) return;
    const int64_t j0 = sb.p * split;
    const int c0 = D > 0 ? 0 : (int)blockIdx.y * chunk, nc = D > 0 ? D : min(chunk, Dm - c0);
    const int metric = D > 0 ? M : kc.metric;
    const OwnPoint<M, D> own(xs.p + i * xs.point, xs.coord, Dm, kc);
    double s0 = 0.0, s1[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) s1[k] = 0.0;
    const double off = offset_weights(
        own, Dm, cA, yc, gA, j0, min(kc.m, j0 + split),
        [&](int sh) {
            s0 = ldexp(s0, sh);
#pragma unroll
            for (int k = 0; k < KC; ++k) s1[k] = ldexp(s1[k], sh);
        },
        [&](const auto& q, const auto&, int64_t j) {
            constexpr int U = sizeof(q) / sizeof(double);
#pragma unroll
            for (int u = 0; u < U; ++u) s0 += q[u];
            add_derivatives<D, KC, U>(metric, Dm, c0, nc, q, own, yc + j * Dm, s1);
        });
    double* o = part + (sb.p * kc.n + i) * (Dm + 2);
    if (c0 == 0) {
        o[0] = off;
        o[1] = s0;
    }
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (k < nc) o[2 + c0 + k] = s1[k];
}

// ---------------------------------------------------------------------------
// Adjoint with respect to the target points: per column j, with
// X_ij = w_i 2^(cfac (k_i + P_ij) + g_j) (the column sweep's terms of X^t, w_i = r_i),
// partial sums S0_j, S1_j (d values) such that grad_y_j = 2 s (S0_j y~_j - S1_j):
//   squared Euclidean (dC/dy = 2 s (y - x)):  S0 = sum_i X_ij,  S1 = sum_i X_ij x~_i;
//   l1 (dC/dy_k = -s sign(x_k - y_k)):      S0 = 0,  S1_k = 1/2 sum_i X_ij sign(x_ik - y_k);
//   l_inf: the same on the coordinate of the largest |x_k - y_k| (first on ties).
// part: [P][m][D+1] partial sums over row splits.
// ---------------------------------------------------------------------------
// One row's data for the column-side adjoint: x~_i in FP64 (dot product), the row's exponent
// term cfac k_i, x~_i in FP32 (S1) and the weight w_i, read with a few wide scalar loads.
template <int D>
struct alignas(16) AdjRow {
    double x[D];
    double ck;
    float xf[D];
    float w;
};

template <int D>
__global__ void adjoint_y_pack(int64_t n, double cA, const double* __restrict__ xc, const float* __restrict__ xcf,
                               const RowVar* __restrict__ rowvar, AdjRow<D>* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    AdjRow<D> a;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        a.x[k] = xc[i * D + k];
        a.xf[k] = xcf[i * D + k];
    }
    const RowVar rv = rowvar[i];
    a.ck = cA * rv.k;
    a.w = rv.wA;
    out[i] = a;
}

template <int M, int D>
__global__ __launch_bounds__(BLOCK) void adjoint_y_sweep(Consts kc, double cA, const AdjRow<D>* __restrict__ rows,
                                                         const double* __restrict__ yc,
                                                         const double* __restrict__ gA,
                                                         double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.n, split);
    const int64_t j = sb.bx * BLOCK + threadIdx.x;
    const int64_t p = sb.p;
    const int64_t i0 = p * split;
    const int64_t i1 = min(kc.n, i0 + split);
    const int64_t jj = j < kc.m ? j : kc.m - 1;
    double y[D];
#pragma unroll
    for (int k = 0; k < D; ++k) y[k] = yc[jj * D + k];
    // e_ij = cfac (G_j + P_ij) + cfac k_i with G_j = g_j / cfac: the dot product starts from
    // the lane's term and the row's term enters as the scalar addend of the exponent FMA
    const double G = gA[jj] / cA;
    double s0 = 0.0, s1[D];
#pragma unroll
    for (int k = 0; k < D; ++k) s1[k] = 0.0;
    auto term = [&](int64_t i, float& a0, float (&a1)[D]) {
        const AdjRow<D>& rw = rows[i];
        const double* xi = rw.x;
        const double dot = pair_term<M, D>(y, xi, G);   // P is symmetric
        const float xij = rw.w * fexp2(fma_su(dot, cA, rw.ck));
        if constexpr (M == METRIC_SQEUCLID) {
            a0 += xij;
#pragma unroll
            for (int k = 0; k < D; ++k) a1[k] = fmaf(xij, rw.xf[k], a1[k]);
        } else if constexpr (M == METRIC_L1) {
#pragma unroll
            for (int k = 0; k < D; ++k) a1[k] = fmaf(0.5f * xij, sgnf(xi[k] - y[k]), a1[k]);
        } else {
            int ks = 0;
            double best = -1.0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const double t = fabs(xi[k] - y[k]);
                if (t > best) {
                    best = t;
                    ks = k;
                }
            }
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (k == ks) a1[k] = fmaf(0.5f * xij, sgnf(xi[k] - y[k]), a1[k]);
        }
    };
    const int64_t nfull = (i1 - i0) / UNROLL;
    for (int64_t c = 0; c <= nfull; ++c) {
        const int64_t ib = i0 + c * UNROLL;
        float a0 = 0.f, a1[D];
#pragma unroll
        for (int k = 0; k < D; ++k) a1[k] = 0.f;
        if (c < nfull) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) term(ib + u, a0, a1);
        } else {
            for (int64_t i = ib; i < i1; ++i) term(i, a0, a1);
        }
        s0 += (double)a0;
#pragma unroll
        for (int k = 0; k < D; ++k) s1[k] += (double)a1[k];
    }
    if (j < kc.m) {
        double* o = part + (p * kc.m + j) * (D + 1);
        o[0] = s0;
#pragma unroll
        for (int k = 0; k < D; ++k) o[1 + k] = s1[k];
    }
}

// The same for the dimensions without a packed form, chunks as in adjoint_sweep_any: the coupling's terms
// X_ij = w_i 2^(cfac (k_i + P_ij) + g_j), every sum FP64.
template <int M, int D, int KC>
__global__ __launch_bounds__(BLOCK) void adjoint_y_sweep_any(Consts kc, int Dm, int chunk, double cA, OwnPts ys,
                                                             const double* __restrict__ xc,
                                                             const double* __restrict__ gA,
                                                             const RowVar* __restrict__ rowvar,
                                                             double* __restrict__ part, int64_t split) {
    const SweepBlock sb = sweep_block(kc.n, split);
    const int64_t j = sb.bx * BLOCK + threadIdx.x;
    if (j >= kc.m) return;
    const int64_t i1 = min(kc.n, (sb.p + 1) * split);
    const int c0 = D > 0 ? 0 : (int)blockIdx.y * chunk, nc = D > 0 ? D : min(chunk, Dm - c0);
    const int metric = D > 0 ? M : kc.metric;
    const OwnPoint<M, D> own(ys.p + j * ys.point, ys.coord, Dm, kc);
    const double g = gA[j];
    double s0 = 0.0, s1[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) s1[k] = 0.0;
    auto run = [&](auto cnt, int64_t i) {
        constexpr int U = decltype(cnt)::value;
        double w[U];
        if constexpr (U == 1) w[0] = own.pair(xc + i * Dm);
        else own.pairs(xc + i * Dm, w);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const RowVar rv = rowvar[i + u];
            w[u] = (double)rv.wA * (double)fexp2(fma(cA, rv.k + w[u], g));
            if (metric == METRIC_SQEUCLID) s0 += w[u];
        }
        add_derivatives<D, KC, U>(metric, Dm, c0, nc, w, own, xc + i * Dm, s1);
    };
    int64_t i = sb.p * split;
    for (; i + UNROLL <= i1; i += UNROLL) run(std::integral_constant<int, UNROLL>{}, i);
    for (; i < i1; ++i) run(std::integral_constant<int, 1>{}, i);
    double* o = part + (sb.p * kc.m + j) * (Dm + 1);
    if (c0 == 0) o[0] = s0;
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (k < nc) o[1 + c0 + k] = s1[k];
}

// A thread takes one coordinate (point e / D, coordinate e % D) a turn: neighbouring threads read
// neighbouring doubles of a partial.
__global__ __launch_bounds__(64) void adjoint_y_finish(Consts kc, int D, int P, double scale,
                                                       const double* __restrict__ yc,
                                                       const double* __restrict__ part, float* __restrict__ grad) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < kc.m * D; e += step) {
        const int64_t j = e / D, k = e % D;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll 16
        for (int p = 0; p < P; ++p) {
            const double* o = part + ((int64_t)p * kc.m + j) * (D + 1);
            s0 += o[0];
            s1 += o[1 + k];
        }
        grad[e] = (float)(scale * (s0 * yc[e] - s1));
    }
}

__global__ __launch_bounds__(64) void adjoint_finish(Consts kc, int D, int P, double scale,
                                                     const double* __restrict__ xc, const double* __restrict__ r,
                                                     const double* __restrict__ part, float* __restrict__ grad) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    const int W = D + 2;
    const double cx = kc.metric == METRIC_SQEUCLID ? 1.0 : 0.0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < kc.n * D; e += step) {
        const int64_t i = e / D, k = e % D;
        const double off = common_offset(part, P, kc.n, W, i);
        double s0 = 0.0, s1 = 0.0;
#pragma unroll 16
        for (int p = 0; p < P; ++p) {
            const double* o = part + ((int64_t)p * kc.n + i) * W;
            s0 += at_offset(o[0], o[1], off);
            s1 += at_offset(o[0], o[2 + k], off);
        }
        grad[e] = (float)(scale * r[i] * (cx * xc[e] - s1 / s0));
    }
}

}  // namespace lampk
