// Batching form: many independent problems advance together, each phase of the
// iteration launched once for all of them.  Each sweep is a persistent loop of a
// machine-sized grid over one work list of (problem, tile) items of every dimension; an
// item runs the same device body as the single-problem kernels, compiled for its problem's
// dimension, with that problem's descriptor.  Sweep items are handed out by an atomic
// counter, largest first.  Every problem keeps its own control block, so a problem that
// meets its tolerance stops (its items exit at once) while the others continue; the host
// then hands its share of the sweep blocks to the problems still running.
#pragma once

#include "lamp_kernels.hpp"

namespace lampk {

struct ProbDesc {
    Ctrl* ctrl;
    Consts kc;
    int32_t d, P_r, P_c, n_dual_blocks;
    int64_t split_r, split_c;
    const double *xc, *yc, *xn2, *yn2, *r, *c;
    double2* gtab;
    double* H;
    RowVar* rowvar;
    double2* rowck;
    double2* rpart;
    double2* cpart;
    DualBufs buf;
    double* respart;
    // set-up
    const float *x, *y;
    double* aux;            // per-column terms of the cost maximum, then of the offsets
    double* stats;          // marginal_stats of r and c, then the cost maximum
    int32_t needs_max, pad;
};

constexpr int BATCH_STATS = 7;   // doubles a problem

struct Item {
    int32_t prob, bx, by, pad;
};

// Every dimension the single-problem sweeps compile for the squared Euclidean cost.
#define LAMP_BATCH_D(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
constexpr int BATCH_MAX_D = 16;

// The descriptor's pointers are loaded from memory, so the compiler cannot tell their
// address space (it would use flat loads) nor that the column data are read-only during
// the sweep.  Re-typing them restores what the single-problem kernels get from their
// arguments: the streamed column data go through the constant address space (scalar
// loads when the address is wave-uniform), per-lane data through the global one.
// (Through an integer: a direct generic -> specific -> generic cast is folded away.)
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
    return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;
}
template <typename T>
__device__ __forceinline__ const T* as_const(const T* p) {
    return (const T*)(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// ---------------------------------------------------------------------------
// Set-up of every problem with d <= BATCH_MAX_D, each step one launch for all of them (a launch per
// problem and step ran 64 problems of 512 to 8192 points through 512 small kernels).  The point and
// column steps take the items of the row finish and dual update, the passes over all pairs those of
// the row sweep, whose partials' room holds their minima.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void batch_marginals(const ProbDesc* __restrict__ pd) {
    const ProbDesc& P = pd[blockIdx.x / 2];
    if (blockIdx.x % 2 == 0) marginal_stats_body(as_global(P.r), P.kc.n, P.stats);
    else marginal_stats_body(as_global(P.c), P.kc.m, P.stats + 3);
}

__global__ __launch_bounds__(BLOCK) void batch_prep(const ProbDesc* __restrict__ pd, const Item* __restrict__ rows,
                                                    int n_rows, const Item* __restrict__ cols) {
    const bool row = (int)blockIdx.x < n_rows;
    const Item it = row ? rows[blockIdx.x] : cols[blockIdx.x - n_rows];
    const ProbDesc& P = pd[it.prob];
    if (P.d > BATCH_MAX_D) return;
    const int64_t i = (int64_t)it.bx * BLOCK + threadIdx.x;
    if (row) {
        if (i == 0) P.stats[BATCH_STATS - 1] = 0.0;
        if (i < P.kc.n) prep_point(P.x, i, P.d, P.x, P.y, const_cast<double*>(P.xc), const_cast<double*>(P.xn2), nullptr, METRIC_SQEUCLID);
    } else if (i < P.kc.m) {
        prep_point(P.y, i, P.d, P.x, P.y, const_cast<double*>(P.yc), const_cast<double*>(P.yn2), nullptr, METRIC_SQEUCLID);
        P.aux[i] = -0.5 * P.yn2[i];
    }
}

// Partial minima of a_j + sgn x~_i . y~_j: sgn = 1 for the cost maximum, -1 for the offsets.
__global__ __launch_bounds__(BLOCK) void batch_extreme(const ProbDesc* __restrict__ pd,
                                                       const Item* __restrict__ items, double sgn) {
    const Item it = items[blockIdx.x];
    const ProbDesc& P = pd[it.prob];
    const int64_t wave_row = (int64_t)it.bx * BLOCK + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    if (wave_row >= P.kc.n || (sgn > 0.0 && !P.needs_max)) return;
    const double* xc = as_global(P.xc);
    const double* yc = as_const(P.yc);
    const double* a = as_const(static_cast<const double*>(P.aux));
    double* part = as_global(reinterpret_cast<double*>(P.rpart));
    switch (P.d) {
#define CASE(D)                                                                                           \
    case D: row_extreme_body<METRIC_SQEUCLID, D>(P.kc, xc, yc, a, sgn, part, P.split_r, it.bx, it.by, 0); break;
        LAMP_BATCH_D(CASE)
#undef CASE
    }
}

__global__ __launch_bounds__(BLOCK) void batch_extreme_max(const ProbDesc* __restrict__ pd,
                                                           const Item* __restrict__ rows) {
    const Item it = rows[blockIdx.x];
    const ProbDesc& P = pd[it.prob];
    if (P.d > BATCH_MAX_D || !P.needs_max) return;
    row_extreme_max_body(P.kc.n, as_global(reinterpret_cast<const double*>(P.rpart)), P.P_r, as_global(P.xn2), nullptr,
                         reinterpret_cast<unsigned long long*>(P.stats + BATCH_STATS - 1),
                         (int64_t)it.bx * BLOCK + threadIdx.x);
}

__global__ __launch_bounds__(BLOCK) void batch_col_table(const ProbDesc* __restrict__ pd,
                                                         const Item* __restrict__ cols,
                                                         const Sched* __restrict__ sched) {
    const Item it = cols[blockIdx.x];
    const ProbDesc& P = pd[it.prob];
    const int64_t j = (int64_t)it.bx * BLOCK + threadIdx.x;
    const int64_t t = P.ctrl->t;
    if (j < P.kc.m)
        col_table_entry(P.kc, sched[t - P.ctrl->t_base], t, j, as_global(P.yn2), as_global(P.buf.nu[t & 1]),
                        as_global(P.buf.theta[t & 1]), as_global(P.gtab), nullptr, 0, as_global(P.aux));
}

__global__ __launch_bounds__(BLOCK) void batch_offsets(const ProbDesc* __restrict__ pd,
                                                       const Item* __restrict__ rows) {
    const Item it = rows[blockIdx.x];
    const ProbDesc& P = pd[it.prob];
    const int64_t i = (int64_t)it.bx * BLOCK + threadIdx.x;
    if (P.d <= BATCH_MAX_D && i < P.kc.n)
        P.H[i] = merge_minima(as_global(reinterpret_cast<const double*>(P.rpart)), P.P_r, P.kc.n, i);
}

// The iterate every problem ended on into the caller's state, where it lies in the other buffer.
__global__ __launch_bounds__(BLOCK) void batch_commit(const ProbDesc* __restrict__ pd, const Item* __restrict__ cols,
                                                      int64_t t0) {
    const Item it = cols[blockIdx.x];
    const ProbDesc& P = pd[it.prob];
    const int64_t j = (int64_t)it.bx * BLOCK + threadIdx.x;
    const int64_t t = P.ctrl->done ? P.ctrl->t_done : P.ctrl->t;
    if (j >= P.kc.m || (t & 1) == (t0 & 1)) return;
    P.buf.nu[t0 & 1][j] = P.buf.nu[t & 1][j];
    P.buf.theta[t0 & 1][j] = P.buf.theta[t & 1][j];
}

// Work items of a persistent sweep: block b starts on item b of the list (largest first, so the
// tail is short) and draws every further one from the phase's counter, one atomic increment a
// block, asked for before the item in hand is swept, so that its latency is hidden.  The counter is
// returned to zero by the next phase kernel of the iteration.
template <typename F>
__device__ __forceinline__ void for_items(unsigned* counter, int n_items, F&& sweep) {
    __shared__ int next_sh[2];
    int k = blockIdx.x;
    for (int half = 0; k < n_items; half ^= 1) {
        unsigned drawn = 0;
        if (threadIdx.x == 0) drawn = atomicAdd(counter, 1u);
        sweep(k);
        if (threadIdx.x == 0) next_sh[half] = (int)(gridDim.x + drawn);
        __syncthreads();
        k = __builtin_amdgcn_readfirstlane(next_sh[half]);   // block-uniform; the halves alternate,
    }                                                        // so one barrier an item is enough
}

__device__ __forceinline__ void reset_counter(unsigned* counter) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;
}

// True in every thread if no problem of the batch runs any more: the iterations queued past the
// last stop leave here instead of drawing every item off the counter (188 us a sweep for the
// 8000 items of 64 problems of 512 to 8192 points).
__device__ __forceinline__ bool batch_idle(const ProbDesc* __restrict__ pd, int count) {
    int running = 0;
    for (int p = threadIdx.x; p < count; p += BLOCK) running |= !halted(pd[p].ctrl);
    return !__syncthreads_or(running);
}

// Row sweep items of every running problem.  What does not depend on the dimension stands outside
// the switch, which holds the bare loops over the streamed points: with the whole body in each of
// its 17 cases 311 scalar registers were spilled (662 in the column sweep, whose vector registers
// for them left room for 5 of 8 waves).  A wave whose rows all lie past the end skips its item.
__global__ __launch_bounds__(BLOCK) void batch_row_sweep(const ProbDesc* __restrict__ pd,
                                                         const Item* __restrict__ items,
                                                         const int* __restrict__ n_active,
                                                         const Sched* sched, unsigned* counter, int count) {
    const int n_items = *n_active;   // items of problems still running (rewritten by the host)
    if ((int)blockIdx.x >= n_items || batch_idle(pd, count)) return;   // surplus blocks leave at once
    for_items(counter, n_items, [&](int k) {
        const Item it = items[k];
        const ProbDesc& P = pd[it.prob];
        const Ctrl* ctrl = as_const(P.ctrl);
        const int64_t n = P.kc.n;
        const int64_t i = (int64_t)it.bx * BLOCK + threadIdx.x;
        const int64_t wave_row = (int64_t)it.bx * BLOCK + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
        if (halted_row(ctrl) || wave_row >= n) return;
        const int64_t t = ctrl->t_row;
        const Sched sc = sched[t - ctrl->t_base];
        const double cA = 2.0 * P.kc.s * sc.lamA * LOG2E;
        const double cB = 2.0 * P.kc.s * sc.lamB * LOG2E;
        const int64_t j0 = it.by * P.split_r;
        const int64_t j1 = min(P.kc.m, j0 + P.split_r);
        const int64_t ii = i < n ? i : n - 1;
        const double* xi = as_global(P.xc) + ii * P.d;
        const double* yc = as_const(P.yc);
        const double2* g = as_const(P.gtab) + (t & 1) * P.kc.m;
        const double h = as_global(P.H)[ii];
        double sumA = 0.0, sumB = 0.0;
        switch (P.d) {
#define CASE(D)                                                                                  \
    case D: {                                                                                    \
        double x[D];                                                                             \
        for (int q = 0; q < D; ++q) x[q] = xi[q];                                                \
        row_sweep_run<METRIC_SQEUCLID, D, true>(cA, cB, x, h, yc, g, j0, j1, sumA, sumB);              \
        break;                                                                                   \
    }
            LAMP_BATCH_D(CASE)
#undef CASE
            default: row_sweep_run_dyn(P.kc, P.d, cA, cB, xi, h, yc, g, j0, j1, sumA, sumB);
        }
        if (i < n) as_global(P.rpart)[it.by * n + i] = make_double2(sumA, sumB);
    });
}

__global__ __launch_bounds__(BLOCK) void batch_row_finish(const ProbDesc* __restrict__ pd,
                                                          const Item* __restrict__ items, int n_items,
                                                          const Sched* sched, unsigned* counter) {
    reset_counter(counter);   // the row sweep of this iteration is complete
    for (int k = blockIdx.x; k < n_items; k += gridDim.x) {
        const Item it = items[k];
        const ProbDesc& P = pd[it.prob];
        row_finish_body(P.ctrl, sched, P.kc, P.d, P.xc, P.yc, P.gtab, P.r, P.xn2, P.rpart, P.P_r, P.H, P.rowvar,
                        P.rowck, nullptr, nullptr, RowVarF32{nullptr, 0}, P.ctrl->done, it.bx);
    }
}

// Column sweep items of every running problem, as the row sweep.
__global__ __launch_bounds__(BLOCK) void batch_col_sweep(const ProbDesc* __restrict__ pd,
                                                         const Item* __restrict__ items,
                                                         const int* __restrict__ n_active,
                                                         const Sched* sched, unsigned* counter, int count) {
    const int n_items = *n_active;   // items of problems still running (rewritten by the host)
    if ((int)blockIdx.x >= n_items || batch_idle(pd, count)) return;   // surplus blocks leave at once
    for_items(counter, n_items, [&](int k) {
        const Item it = items[k];
        const ProbDesc& P = pd[it.prob];
        const Ctrl* ctrl = as_const(P.ctrl);
        const int64_t m = P.kc.m;
        const int64_t j = (int64_t)it.bx * BLOCK + threadIdx.x;
        const int64_t wave_col = (int64_t)it.bx * BLOCK + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
        if (halted(ctrl) || wave_col >= m) return;
        const int64_t t = ctrl->t;
        const Sched sc = sched[t - ctrl->t_base];
        const double cA = 2.0 * P.kc.s * sc.lamA * LOG2E;
        const double cB = 2.0 * P.kc.s * sc.lamB * LOG2E;
        const int64_t i0 = it.by * P.split_c;
        const int64_t i1 = min(P.kc.n, i0 + P.split_c);
        const int64_t jj = j < m ? j : m - 1;
        const double* yj = as_global(P.yc) + jj * P.d;
        const double* xc = as_const(P.xc);
        const double2* rowck = as_const(P.rowck);
        const double2 g = as_global(P.gtab)[(t & 1) * m + jj];
        const double G = g.y / cB;
        const double Dj = g.x - cA * G;
        const bool factor = P.kc.factor_cols;
        double sumA = 0.0, sumB = 0.0;
        switch (P.d) {
#define CASE(D)                                                                                      \
    case D: {                                                                                        \
        double y[D];                                                                                 \
        for (int q = 0; q < D; ++q) y[q] = yj[q];                                                    \
        if (factor) col_sweep_run<METRIC_SQEUCLID, D, true, true>(cA, cB, y, G, Dj, xc, rowck, i0, i1, sumA, sumB); \
        else col_sweep_run<METRIC_SQEUCLID, D, false, true>(cA, cB, y, G, Dj, xc, rowck, i0, i1, sumA, sumB);       \
        break;                                                                                       \
    }
            LAMP_BATCH_D(CASE)
#undef CASE
            default: col_sweep_run_dyn(P.kc, P.d, cA, cB, yj, G, Dj, xc, rowck, i0, i1, sumA, sumB);
        }
        const double inv_n = 1.0 / (double)P.kc.n;   // the row weights r_i enter as n r_i (rowck)
        sumA *= factor ? exp2(Dj) * inv_n : inv_n;
        sumB *= inv_n;
        if (j < m) as_global(P.cpart)[it.by * m + j] = make_double2(sumA, sumB);
    });
}

__global__ __launch_bounds__(BLOCK) void batch_dual_update(const ProbDesc* __restrict__ pd,
                                                           const Item* __restrict__ items, int n_items,
                                                           const Sched* sched, unsigned* counter) {
    reset_counter(counter);   // the column sweep of this iteration is complete
    for (int k = blockIdx.x; k < n_items; k += gridDim.x) {
        const Item it = items[k];
        const ProbDesc& P = pd[it.prob];
        dual_update_body(P.ctrl, sched, P.kc, P.cpart, P.P_c, P.c, P.yn2, P.buf, P.gtab, nullptr, 0, P.respart,
                         TraceCols{nullptr, nullptr, nullptr, nullptr}, nullptr, it.bx);
    }
}

// Block p completes the iteration of problem p (residual, stop decision, t + 1).
__global__ __launch_bounds__(BLOCK) void batch_dual_finish(const ProbDesc* __restrict__ pd, const Sched* sched) {
    const ProbDesc& P = pd[blockIdx.x];
    complete_iteration<BLOCK>(P.ctrl, sched, P.respart, nullptr, P.n_dual_blocks);
}

}  // namespace lampk
