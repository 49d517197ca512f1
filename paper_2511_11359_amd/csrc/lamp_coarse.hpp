// The cost maximum and the exact row offsets of the squared Euclidean cost at d > 16, both
//     out_i = min_j (a_j + sgn x~_i . y~_j),
// with INT8 matrix cores finding the few tiles that hold a minimum and FP64 matrix cores
// evaluating those.  The FP64 product of every pair costs 14.6 ms at n = m = 2^16, d = 64 (the
// FP64 matrix cores run at 1/64 of the INT8 rate); only one pair in thousands decides a minimum.
//
// A centred coordinate is a 22-bit fixed-point integer X = round(x~ 2^f) in three signed
// base-256 digits, and six of the nine digit products are kept, each level exact in the INT32
// accumulators of v_mfma_i32_16x16x64_i8:
//     X . Y = 2^32 L_0 + 2^24 L_1 + 2^16 L_2 + ...,   L_l = sum_{i+j=l} X_i . Y_j.
// The levels left out and the rounding of the coordinates are bounded by coarse_error below, so
// a minimum can only lie where the coarse value is within twice that bound of the coarse minimum.
// Those 16 x 16 tiles are evaluated with the FP64 instructions, operands and order of
// row_extreme_mfma64, so that the result is the same to the last bit.
//
// That pays where few tiles are near a minimum.  One point 100 times as far out as the others (the digits'
// unit follows the largest coordinate), one-hot features or points that repeat put most tiles near one, and
// evaluating those tile by tile takes 2.2 times the FP64 pass.  So each pass watches what it meets
// (CoarseWatch), blocks that start after enough was seen leave at once, and row_extreme_mfma64 runs
// instead, on the device's own word for the offsets and after the host's wait for the maximum.  One step /
// the maximum, tile by tile -> given up, against the FP64 pass from the start: one-hot 65536 x 65536 x 64
// 52.1 -> 32.7 (32.5) / 16.6 -> 15.5 (15.0) ms, x 24 26.5 -> 18.2 (17.9) / 9.3 -> 8.3 (7.8), 8192 x 8192 x 64
// 0.98 -> 0.79 (0.78) / 0.45 (0.38); an outlier, 40000 x 30000 x 100 31.0 -> 18.6 (18.5) / 1.1 (8.6).
//
// Per pair of points: 6 KP / 64 x 16 matrix cycles a 16 x 16 tile and 6 vector slots (a shift, two
// conversions, two FMAs, a minimum or a comparison): at 2^16, d = 64 1.7 ms a pass, 2.4 ms with the
// FP64 tiles of the offsets, 33 us for the FP64 tiles of the maximum.
#pragma once

#include "lamp_mfma.hpp"

namespace lampk {

constexpr int COARSE_DIGITS = 3;

// Scalars of one use of the coarse passes, cleared by launch_digits.
struct CoarseWatch {
    unsigned long long max;   // refine_max's result (bits)
    unsigned long long top;   // the largest row value of the blocks that have finished (bits)
    int tiles;                // row tiles that can hold the maximum
    int bad;                  // a coordinate without digits
    int many;                 // too many near tiles: the coarse passes are given up
    int pairs;                // first pass, offsets: near pairs in the near tiles
    // of the reporting blocks, counts in the halves of a word: those seen above, the near ones below
    unsigned long long first;    // row tiles (offsets) or waves (maximum) of the first pass
    unsigned long long second;   // waves of the second pass, those that meet near tiles most of the time
};

__device__ __forceinline__ bool given_up(const int* many) {
    return __hip_atomic_load(many, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
__device__ __forceinline__ void give_up(int* many) {
    __hip_atomic_store(many, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Adds to one of the counts; the total.  Every atomic on a word takes its turn, 10 to 20 ns (6256 blocks with
// three each: 0.35 ms), so that only the blocks of up to about 256 in the grid report (reporting), in rows of P
// splits spread over it.
struct Count {
    unsigned near, seen;
};
__device__ __forceinline__ Count count_in(unsigned long long* word, unsigned near, unsigned seen) {
    const unsigned long long v = ((unsigned long long)seen << 32) | near, t = atomicAdd(word, v) + v;
    return Count{(unsigned)t, (unsigned)(t >> 32)};
}
__device__ __forceinline__ bool reporting(int P) { return blockIdx.x / P % max(1u, gridDim.x / 256) == 0; }

__device__ __forceinline__ i32x4 mma_i8(i32x4 a, i32x4 b, i32x4 c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// 2^f = 2^14 times the range scale 2^(7-e) (2^e <= max |coordinate| < 2^(e+1)): |X| < 2^22.
constexpr double COARSE_SCALE = 0x1p14;

// 2^-2f.
__device__ __forceinline__ double coarse_unit(const double* __restrict__ range) {
    const double f = *range * COARSE_SCALE;
    return 1.0 / (f * f);
}

// Bound on the error of a coarse inner product: per coordinate two products of level 3 and one
// of level 4, of at most 2^14 each, and the two roundings (half a unit times 2^22).
__device__ __forceinline__ double coarse_error(const double* __restrict__ range, int d) {
    return 1.01 * (double)d * (0x1p23 + 0x1p14 + 0x1p22) * coarse_unit(range);
}

// Digit planes out[point][digit][KP], zero padded to KP coordinates and cnt_pad points; a thread
// writes four coordinates of every digit.  A coordinate that is not finite has no digits: it
// raises *bad, and the FP64 products of every pair are taken instead.
__global__ void prep_digits(const double* __restrict__ src, int64_t cnt, int d, int KP, int64_t cnt_pad,
                            const double* __restrict__ range, int8_t* __restrict__ out, int* __restrict__ bad) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int quads = KP / 4;
    if (idx >= cnt_pad * quads) return;
    const int64_t i = idx / quads;
    const int k0 = (int)(idx % quads) * 4;
    const double f = *range * COARSE_SCALE;
    uint32_t pack[COARSE_DIGITS] = {};
    for (int q = 0; q < 4; ++q) {
        const int k = k0 + q;
        double x = (i < cnt && k < d) ? src[i * d + k] * f : 0.0;
        if (!(fabs(x) <= 0x1p22)) {
            *bad = 1;
            x = 0.0;
        }
        int v = (int)rint(x);
#pragma unroll
        for (int g = COARSE_DIGITS - 1; g >= 0; --g) {
            const int dig = g ? (int)(int8_t)(v & 255) : v;   // |v| <= 64 at the top digit
            pack[g] |= (uint32_t)(uint8_t)dig << (8 * q);
            v = (v - dig) >> 8;
        }
    }
#pragma unroll
    for (int g = 0; g < COARSE_DIGITS; ++g)
        *reinterpret_cast<uint32_t*>(out + (i * COARSE_DIGITS + g) * KP + k0) = pack[g];
}

__global__ void clear_words(int cnt, int* __restrict__ w) {
    if ((int)threadIdx.x < cnt) w[threadIdx.x] = 0;
}

// A tile of 16 points in LDS: digit rows padded by 16 bytes (the 16-byte reads of 8 rows then
// cover all 32 banks), the columns' a_j behind them in 16-byte slots.
template <int KP>
struct CoarseTile {
    static constexpr int ROW_BYTES = COARSE_DIGITS * KP;
    static constexpr int STRIDE = ROW_BYTES + 16;
    static constexpr int TILE_BYTES = 16 * ROW_BYTES;
    static constexpr int CHUNKS = TILE_BYTES / 16;
    static constexpr int PER_THREAD = (CHUNKS + BLOCK - 1) / BLOCK;
    static constexpr int BUF = 16 * STRIDE + 16 * 16;
    static_assert(PER_THREAD <= 4, "tile larger than the prefetch registers");
};

template <int KP>
__device__ __forceinline__ void coarse_fetch(const TileSrc& src, int tile, TileRegs& R) {
    using L = CoarseTile<KP>;
    const uint32_t tile_off = (uint32_t)tile * (uint32_t)L::TILE_BYTES;
    unroll_for<0, L::PER_THREAD>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const uint32_t c = threadIdx.x + q * BLOCK;
        constexpr bool full = (q + 1) * BLOCK <= L::CHUNKS;   // every thread has a piece
        if (full || c < (uint32_t)L::CHUNKS)
            treg<q>(R) = __builtin_amdgcn_raw_buffer_load_b128(src.ops, c * 16u, tile_off, 0);
    });
    const i32x2 v = __builtin_amdgcn_raw_buffer_load_b64(src.scal, (threadIdx.x & 15u) * 8u, (uint32_t)tile * 128u, 0);
    R.s = i32x4{v.x, v.y, 0, 0};
}

template <int KP>
__device__ __forceinline__ void coarse_store(char* lds, TileRegs& R) {
    using L = CoarseTile<KP>;
    store_tile<16, L::ROW_BYTES, L::STRIDE, L::PER_THREAD>(lds, R);
}

// The digits of one point for this lane: lane group g (lane / 16) supplies coordinates
// [64 s + 16 g, 64 s + 16 g + 16) of instruction s.
template <int KP>
struct Digits {
    i32x4 v[COARSE_DIGITS][KP / 64];
    __device__ __forceinline__ void load(const char* row, int grp) {
#pragma unroll
        for (int g = 0; g < COARSE_DIGITS; ++g)
#pragma unroll
            for (int s = 0; s < KP / 64; ++s)
                v[g][s] = *reinterpret_cast<const i32x4*>(row + g * KP + s * 64 + grp * 16);
    }
};

// c + L_LEVEL.  |L_l| <= 3 KP 2^14, so (L_0 << 8) + L_1 fits 31 bits for KP <= 128.
template <int KP, int LEVEL>
__device__ __forceinline__ i32x4 digit_level(const Digits<KP>& a, const Digits<KP>& b, i32x4 c) {
    unroll_for<0, COARSE_DIGITS>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = LEVEL - i;
        if constexpr (j >= 0 && j < COARSE_DIGITS) {
#pragma unroll
            for (int s = 0; s < KP / 64; ++s) c = mma_i8(a.v[i][s], b.v[j][s], c);
        }
    });
    return c;
}

// Row tiles of 16 points a wave owns.
constexpr int coarse_rows(int KP) { return KP <= 64 ? 4 : 2; }

// PICK = false: part[p][i] = the coarse minimum of row i over the column tiles of split p.
// PICK = true: the FP64 minimum of row i over the tiles of the split in which some row of the
// wave's row tile may hold its minimum (coarse[i]: the coarse minimum over every split), +inf if
// there is none; the merge over the splits then gives the minimum.  Lane c16 holds column
// 16 jt + c16 of tile jt, register r row 4 g + r (g = lane / 16) of the integer products and row
// 4 r + g of the FP64 ones.
// xn2: the squared norms for the cost maximum, null for the offsets (what a finished split is asked).
template <int KP, int KP64, bool PICK>
__global__ __launch_bounds__(BLOCK, 2) void row_extreme_coarse(Consts kc, int d, const int8_t* __restrict__ xop,
                                                               const int8_t* __restrict__ yop,
                                                               const double* __restrict__ range,
                                                               const double* __restrict__ aj, double sgn,
                                                               const double* __restrict__ coarse,
                                                               const double* __restrict__ xn2, CoarseWatch* watch,
                                                               const double* __restrict__ xop64,
                                                               const double* __restrict__ yop64,
                                                               double* __restrict__ part, int64_t tiles_per_split,
                                                               int P, int64_t m_tiles, int64_t n_tiles) {
    using L = CoarseTile<KP>;
    constexpr int RT = coarse_rows(KP);
    constexpr int NS64 = KP64 / 4;
    __shared__ __align__(16) char lds[2][L::BUF];
    __shared__ int stop[3];   // by the parity of the group of tiles, and at the start
    const double unit = sgn * coarse_unit(range);
    const double whi = unit * 0x1p24, wmid = unit * 0x1p16;
    const int lane = threadIdx.x & 63;
    const int grp = lane >> 4, c16 = lane & 15;
    const int64_t b = blockIdx.x;
    const int p = (int)(b % P);
    const int64_t rt0 = ((b / P) * 4 + (threadIdx.x >> 6)) * RT;   // first row tile of the wave
    const int jt0 = (int)((int64_t)p * tiles_per_split);
    const int jt1 = (int)min(m_tiles, (int64_t)jt0 + tiles_per_split);
    if (jt0 >= jt1) return;
    Digits<KP> a[RT];
    double best[RT][4];     // PICK: the FP64 minima
    double limit[RT][4];    // PICK: rows' largest coarse value that can be a minimum
    // a coordinate without digits: every tile is near
    const double slack = watch->bad ? __builtin_inf() : 2.0 * coarse_error(range, d);
#pragma unroll
    for (int u = 0; u < RT; ++u) {
        const int64_t rt = min(rt0 + u, n_tiles - 1);   // row tiles past the end repeat the last, unwritten
        a[u].load(reinterpret_cast<const char*>(xop) + (rt * 16 + c16) * L::ROW_BYTES, grp);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            best[u][r] = __builtin_inf();
            if constexpr (PICK) {
                const int64_t i = rt * 16 + 4 * grp + r;
                limit[u][r] = coarse[i < kc.n ? i : kc.n - 1] + slack;
            }
        }
    }
    const TileSrc src = make_tile_src(yop, (uint32_t)(m_tiles * L::TILE_BYTES), aj, (uint32_t)(kc.m * 8));
    const int jl = jt1 - 1;
    // the digits and a_j of tile jt in LDS buffer q, and the coarse values of the wave's row tile u with it
    auto tile_load = [&](int q, int jt, Digits<KP>& bv, double& aval) {
        bv.load(lds[q] + c16 * L::STRIDE, grp);
        aval = *reinterpret_cast<const double*>(lds[q] + 16 * L::STRIDE + c16 * 16);
        if ((int64_t)jt * 16 + c16 >= kc.m) aval = __builtin_inf();
    };
    auto values = [&](int u, const Digits<KP>& bv, double aval, double (&v)[4]) {
        const i32x4 zero = {0, 0, 0, 0};
        const i32x4 hi = digit_level<KP, 1>(a[u], bv, digit_level<KP, 0>(a[u], bv, zero) << 8);
        const i32x4 mid = digit_level<KP, 2>(a[u], bv, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fma((double)hi[r], whi, fma((double)mid[r], wmid, aval));
    };
    const bool report = reporting(P);
    // of the first pass the blocks past the first 512, which start at once (two a CU), of long splits: a short
    // one would wait for the answer (200000 x 512 x 64 0.78 -> 0.82 ms)
    const bool asks = PICK || (b >= 512 && tiles_per_split >= 32);
    const int quit = asks && threadIdx.x == 0 ? given_up(&watch->many) : 0;   // in flight with the first tile
    TileRegs pf;
    coarse_fetch<KP>(src, jt0, pf);
    coarse_store<KP>(lds[0], pf);
    if (threadIdx.x == 0) {
        stop[0] = stop[1] = 0;
        stop[2] = quit;
        if (PICK && report) count_in(&watch->second, 0, 4);
    }
    __syncthreads();
    if (stop[2]) return;
    int picked = 0;
    bool dense = false;
    // in groups of tiles, between which the block may stop: an inner loop without that question
    for (int g0 = jt0, g1, group = 0; g0 < jt1; g0 = g1, ++group) {
        g1 = min(jt1, g0 + (PICK ? 4 : 32));
        for (int jt = g0; jt < g1; ++jt) {
            const int cur = (jt - jt0) & 1;
            coarse_fetch<KP>(src, min(jt + 1, jl), pf);
            Digits<KP> bv;
            double aval;
            tile_load(cur, jt, bv, aval);
#pragma unroll
            for (int u = 0; u < RT; ++u) {
                double v[4];
                values(u, bv, aval, v);
                bool near = false;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (PICK) near = near || !(v[r] > limit[u][r]);
                    else best[u][r] = fmin(best[u][r], v[r]);
                }
                if constexpr (PICK) {
                    if (__any(near)) {   // a wave at a time: rare where this pays
                        const int64_t rt = min(rt0 + u, n_tiles - 1);
                        const double* ap = xop64 + (rt * 16 + c16) * KP64 + grp * NS64;
                        const double* bp = yop64 + ((int64_t)jt * 16 + c16) * KP64 + grp * NS64;
                        doublex4 dd = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
                        for (int s = 0; s < NS64; ++s) dd = mma64(sgn * ap[s], bp[s], dd);
#pragma unroll
                        for (int q = 0; q < 4; ++q) best[u][q] = fmin(best[u][q], aval + dd[q]);
                        ++picked;
                    }
                }
            }
            if constexpr (PICK) {
                // A near tile costs 2.2 times its share of the FP64 pass (65536 x 65536 x 64, all of them: 31.7 ms
                // against 14.6, after 3.4 ms of coarse passes): above 3/8 of them that pass is the shorter way.
                // A wave that meets as many says so, and stops its block once as many of the reporting waves have.
                if (picked >= 8 && 8 * picked > 3 * RT * (jt - jt0 + 1) && lane == 0) {
                    if (report && !dense) {
                        const Count c = count_in(&watch->second, 1, 0);
                        if (c.near >= 16 && 8 * c.near > 3 * c.seen) give_up(&watch->many);
                    }
                    dense = true;
                    if (given_up(&watch->many)) stop[group & 1] = 1;
                }
            }
            coarse_store<KP>(lds[cur ^ 1], pf);
            __syncthreads();
        }
        if constexpr (PICK) {
            // a group's word is written before its last barrier, the next one's for the other parity: the same in
            // every wave
            if (stop[group & 1]) return;
        } else if (asks && g1 < jt1) {
            if (threadIdx.x == 0) stop[group & 1] = given_up(&watch->many);
            __syncthreads();
            if (stop[group & 1]) return;
        }
    }
    if constexpr (!PICK) {
        // What the split says of the data.  Offsets: whether its last tile, still in LDS, is near the split's minima
        // (more often than near the rows').  Of T tiles 1 - (1 - 1 / T)^16 are by the minima of their 16 rows alone,
        // with 16 / T pairs: 64% and 1 at the fewest asked, 16.  So three in four tiles have to be, with a pair a
        // tile beyond twice that.  Maximum: whether the wave's largest row value ties with that of the blocks before.
        __shared__ double tops[4];
        __shared__ int nears[4], pairs[4];
        // (The maximum only where blocks are still to start and ask: 12000 x 9000 x 24 58 us, 65 with the question.)
        const bool for_max = xn2 != nullptr;
        if (report && (for_max ? gridDim.x > 512 && tiles_per_split >= 32 : jt1 - jt0 >= 16)) {
            Digits<KP> bv;
            double aval, top = 0.0;
            int near_tiles = 0, near_pairs = 0;
            tile_load((jt1 - jt0) & 1, jl, bv, aval);
#pragma unroll
            for (int u = 0; u < RT; ++u) {
                double v[4];
                if (!for_max) values(u, bv, aval, v);
                int cnt = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double m = best[u][r];
#pragma unroll
                    for (int o = 8; o > 0; o >>= 1) m = fmin(m, __shfl_xor(m, o, 64));
                    const int64_t i = (rt0 + u) * 16 + 4 * grp + r;
                    if (for_max) {
                        if (i < kc.n) top = fmax(top, xn2[i] - 2.0 * m);
                    } else {
                        cnt += __popcll(__ballot(i < kc.n && v[r] <= m + slack));
                    }
                }
                near_tiles += cnt > 0;
                near_pairs += cnt;
            }
#pragma unroll
            for (int o = 32; o >= 16; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
            if (lane == 0) {
                tops[threadIdx.x >> 6] = top;
                nears[threadIdx.x >> 6] = near_tiles;
                pairs[threadIdx.x >> 6] = near_pairs;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                unsigned near = nears[0] + nears[1] + nears[2] + nears[3];
                if (for_max) {
                    const double most = fmax(fmax(tops[0], tops[1]), fmax(tops[2], tops[3]));
                    const double old = __longlong_as_double((long long)atomicMax(
                        &watch->top, (unsigned long long)__double_as_longlong(most)));
                    for (int w = 0; w < 4; ++w) near += fabs(tops[w] - old) <= 2.0 * slack;
                }
                int all = pairs[0] + pairs[1] + pairs[2] + pairs[3];
                if (!for_max) all += atomicAdd(&watch->pairs, all);
                const Count c = count_in(&watch->first, near, for_max ? 4 : 4 * RT);
                const bool plenty = for_max || (double)all * tiles_per_split > (32.0 + tiles_per_split) * c.seen;
                if (c.seen >= 128 && 4 * c.near > 3 * c.seen && plenty) give_up(&watch->many);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < RT; ++u) {
        reduce_lanes<4, 8>(best[u], [](double x, double y) { return fmin(x, y); });
        const int r = c16 >> 2;
        const int64_t row = (rt0 + u) * 16 + (PICK ? 4 * r + grp : 4 * grp + r);
        if (c16 % 4 == 0 && row < kc.n && rt0 + u < n_tiles) part[(int64_t)p * kc.n + row] = best[u][0];
    }
}

// The row tiles that can hold the largest value xn2_i - 2 min_i: some row's coarse value (rowmax)
// is within twice its error (twice the product's) of the largest, *top.  Up to COARSE_MAX_TILES
// are listed; watch->tiles goes on counting.
constexpr int COARSE_MAX_TILES = 64;
constexpr int COARSE_MAX_SPLITS = 64;

__global__ void select_max_tiles(int64_t n, int d, const double* __restrict__ rowmax, const double* __restrict__ top,
                                 const double* __restrict__ range, int* __restrict__ list, CoarseWatch* watch) {
    if (watch->many) return;   // the row values are not there
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool near = i < n && rowmax[i] >= *top - 4.0 * coarse_error(range, d);
    const unsigned long long lanes = __ballot(near);   // 64 consecutive rows: 4 tiles of 16
    const int t = threadIdx.x & 63;
    if (t >= 4 || !((lanes >> (16 * t)) & 0xffffull)) return;
    const int k = atomicAdd(&watch->tiles, 1);
    if (k < COARSE_MAX_TILES) list[k] = (int)((i - t) / 16) + t;
}

// watch->max = the largest xn2_i - 2 min_j (a_j + x~_i . y~_j) over the listed row tiles, from the FP64
// matrix cores: wave w of block (k, q) takes column tiles 4 q + w, 4 q + w + 4 COARSE_MAX_SPLITS,
// ... of row tile list[k].  (Non-negative doubles order as their bits do; the rounding of
// xn2 - 2 min is monotone, so the largest of the parts is the row's value.)
template <int KP64>
__global__ __launch_bounds__(BLOCK) void refine_max(Consts kc, const double* __restrict__ xop64,
                                                    const double* __restrict__ yop64,
                                                    const double* __restrict__ xn2, const double* __restrict__ aj,
                                                    const int* __restrict__ list, int64_t m_tiles,
                                                    CoarseWatch* watch) {
    constexpr int NS64 = KP64 / 4;
    const int k = blockIdx.x / COARSE_MAX_SPLITS, q0 = blockIdx.x % COARSE_MAX_SPLITS;
    if (k >= watch->tiles || watch->tiles > COARSE_MAX_TILES) return;
    const int lane = threadIdx.x & 63;
    const int grp = lane >> 4, c16 = lane & 15;
    const int64_t i0 = (int64_t)list[k] * 16;
    double a[NS64];
    const double* ap = xop64 + (i0 + c16) * KP64 + grp * NS64;
#pragma unroll
    for (int s = 0; s < NS64; ++s) a[s] = ap[s];
    double best[4] = {__builtin_inf(), __builtin_inf(), __builtin_inf(), __builtin_inf()};
    for (int64_t jt = q0 * 4 + (threadIdx.x >> 6); jt < m_tiles; jt += 4 * COARSE_MAX_SPLITS) {
        const int64_t j = jt * 16 + c16;
        const double* bp = yop64 + j * KP64 + grp * NS64;
        const double aval = j < kc.m ? aj[j] : __builtin_inf();
        doublex4 dd = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < NS64; ++s) dd = mma64(a[s], bp[s], dd);
#pragma unroll
        for (int q = 0; q < 4; ++q) best[q] = fmin(best[q], aval + dd[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) best[q] = fmin(best[q], __shfl_xor(best[q], o, 64));
        const int64_t row = i0 + 4 * q + grp;
        if (c16 == q && row < kc.n)
            atomicMax(&watch->max, (unsigned long long)__double_as_longlong(fmax(xn2[row] - 2.0 * best[q], 0.0)));
    }
}

}  // namespace lampk
