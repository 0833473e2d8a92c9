// C = A*B row by row (Gustavson's order), for operands whose 16x16 tiles hold too little for block products: a
// (A tile, B tile) pair of a graph or of a mesh with one unknown per node multiplies a handful of entries, and the
// task list, the counting pass and the block products all cost by the pair.  Here everything costs by the
// intermediate product a_ik * b_kj:
//
//   k_row_prepare   one pass over an operand: validation, entries as {column, value} records, tiles per tile-row,
//                   and for A the number of intermediate products of every row
//   k_row_plan      candidate tile pairs (the measure by which tsp_spgemm chooses this path), the lists of work
//   k_row_merge     rows with few, short rows of B behind them: a lane per row of B, merged in column order
//   k_heavy_count   the other rows: a block per row, one bit per column of C in LDS
//   k_heavy_fill    a block per row and some windows of columns, a dense accumulator in LDS
//
// Runs are bit-identical.  Products of fp16 numbers are exact in fp32.  A merged entry is summed by the lanes of its
// group as a tree, in fp32.  A heavy entry is summed in integers where every partial sum is exact in them (all products
// are multiples of a power of two that the operands' values say; then the order of the additions does not matter and a
// whole block shares the accumulator), and otherwise in fp64 by one wave in the order of the entries of A.
#include "common.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace tsp {

constexpr int kMergeProducts = 256;      // a merged row has at most this many intermediate products
constexpr int kPlanBlocks = 128;         // blocks of k_row_plan
constexpr int kPlanSums = 8;
constexpr int kWindow = 4096;            // columns of C per window of the heavy rows (2048 where C is no wider)
constexpr int kSpanWindows = 64;         // windows whose bits the LDS of a block of k_heavy_count holds (32 KB)
constexpr int kGroupWindows = 4;         // tasks begin at a multiple of this many windows
constexpr int kHeavyThreads = 512;
constexpr int32_t kNoCol = 0x7FFFFFFF;
// Intermediate products behind one task of k_heavy_fill (a row, or some of its windows)
constexpr int kTaskProducts = 65536;
constexpr int64_t kRowPairProducts = 64; // products per candidate pair of tiles up to which the rows are the better way

struct RowMatrix {                       // an operand in the form the row kernels read
    int32_t *start = nullptr;            // int32[rows + 1], clamped to [0, nnz]
    int2 *rec = nullptr;                 // per entry {column (clamped), value rounded to fp16, as fp32 bits}
    int32_t *ntiles = nullptr;           // tiles of every tile-row
    int32_t *tile_col = nullptr;         // their columns, at the position of the tile-row's first entry; any order
    uint32_t *range = nullptr;           // magnitude and granularity of every tile-row's values (value_range)
};

template <typename RP, typename VT>
struct PrepareArgs {
    const RP *row_ptr;
    const int32_t *col;
    const VT *val;
    int64_t rows, cols, nnz;
    int bitmap_words;
    int validate;
    RowMatrix out;
    int32_t *ub;                         // products per row (of A), or null
    const void *b_row_ptr;               // of B, as the caller gave it
    int b_is_i64;
    int64_t b_rows, b_nnz;
    int64_t *d_scalars;
};

__device__ __forceinline__ float rounded_value(uint16_t bits) {
    return (float)__builtin_bit_cast(_Float16, bits);
}
__device__ __forceinline__ float rounded_value(float v) { return (float)(_Float16)v; }

// Of a value v != 0: {256 + e} << 16 | {256 - g}, |v| < 2^e and v a multiple of 2^g; infinities and NaNs are as large as
// can be.  The larger of each half over a set of values holds for the set.
__device__ __forceinline__ uint32_t value_range(float v) {
    const uint32_t b = __float_as_uint(v) & 0x7FFFFFFFu;
    if (b == 0) return 0;
    if (b >= 0x7F800000u) return 0x03FF03FFu;
    const int exponent = (int)(b >> 23), low = __ffs((int)((b & 0x7FFFFFu) | 0x800000u)) - 1;
    return (uint32_t)(256 + exponent - 126) << 16 | (uint32_t)(256 - (exponent - 150 + low));
}
__device__ __forceinline__ uint32_t range_max(uint32_t x, uint32_t y) {
    return max(x & 0xFFFF0000u, y & 0xFFFF0000u) | max(x & 0xFFFFu, y & 0xFFFFu);
}

// A team of kTeam threads per tile-row (a wave, or a block of 256 for long tile-rows), its entries flat over the
// lanes.  The team's bitmap over the tile columns tells the first entry that falls into a tile (the atomic returns the
// word before): those lanes list the tile.  Bound by the loads of B's row pointers and by instructions.
template <int kTeam, typename RP, typename VT>
__global__ __launch_bounds__(256) void k_row_prepare(const PrepareArgs<RP, VT> a) {
    constexpr int kTeams = 256 / kTeam;
    extern __shared__ uint32_t lds_bitmap[];
    __shared__ int32_t s_ptr[kTeams][T + 1];
    __shared__ unsigned long long s_ub[kTeams][T];
    __shared__ int32_t s_count[kTeams];
    __shared__ uint32_t s_range[2][kTeams];
    const int team = threadIdx.x / kTeam, tid = threadIdx.x % kTeam, lane = lane_id();
    uint32_t *bitmap = lds_bitmap + team * a.bitmap_words;
    const int64_t tile_rows = (a.rows + T - 1) / T;
    const int64_t I = (int64_t)blockIdx.x * kTeams + team;
    const bool live = I < tile_rows;
    bool bad = false;
    if (live) {
        for (int w = tid; w < a.bitmap_words; w += kTeam) bitmap[w] = 0;
        if (tid <= T) {
            const int64_t i = min(I * T + tid, a.rows);
            const int64_t raw = (int64_t)a.row_ptr[i];
            const int64_t p = min(max(raw, (int64_t)0), a.nnz);
            bad = raw != p || (i == 0 && raw != 0) || (i == a.rows && raw != a.nnz) ||
                  (i < a.rows && (int64_t)a.row_ptr[i + 1] < raw);
            s_ptr[team][tid] = (int32_t)p;
            if (tid < T) s_ub[team][tid] = 0;
            if (i < a.rows ? tid < T : true) a.out.start[i] = (int32_t)p;
        }
        if (tid == 0) {
            s_count[team] = 0;
            s_range[0][team] = s_range[1][team] = 0;
        }
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (live) {
        const int32_t e0 = s_ptr[team][0], e1 = s_ptr[team][T];
        int32_t listed = 0;
        uint32_t range = 0;
        for (int32_t base = e0 + (tid & ~63); base < e1; base += kTeam) {
            const int32_t k = base + lane;
            const bool on = k < e1;
            int r = T;
            int32_t c = 0, len = 0, prev = -1;
            if (on) {
                r = 0;
#pragma unroll
                for (int step = T / 2; step >= 1; step >>= 1)
                    if (s_ptr[team][r + step] <= k) r += step;
                c = a.col[k];
                const float v = rounded_value(a.val[k]);
                if (k > s_ptr[team][r]) {
                    prev = a.col[k - 1];
                    bad = bad || prev >= c;
                }
                if ((uint32_t)c >= (uint64_t)a.cols) {
                    bad = true;
                    c = 0;
                }
                a.out.rec[k] = make_int2(c, (int)__float_as_uint(v));
                range = range_max(range, value_range(v));
                if (a.ub && c < a.b_rows) {
                    int64_t s, e;
                    if (a.b_is_i64) {
                        s = static_cast<const int64_t *>(a.b_row_ptr)[c];
                        e = static_cast<const int64_t *>(a.b_row_ptr)[c + 1];
                    } else {
                        s = static_cast<const int32_t *>(a.b_row_ptr)[c];
                        e = static_cast<const int32_t *>(a.b_row_ptr)[c + 1];
                    }
                    len = (int32_t)min(max(e - s, (int64_t)0), (int64_t)((1 << 25) - 1));
                }
            }
            const int32_t t = c >> 4;
            bool first = on && (prev < 0 || (prev >> 4) != t);
            if (first) {
                const uint32_t bit = 1u << (t & 31);
                first = !(atomicOr(&bitmap[t >> 5], bit) & bit);
            }
            const unsigned long long firsts = __ballot(first);
            int32_t at = listed;
            if constexpr (kTeam == 64) {
                listed += __popcll(firsts);
            } else if (firsts) {
                if (lane == 0) at = atomicAdd(&s_count[team], __popcll(firsts));
                at = __builtin_amdgcn_readfirstlane(at);
            }
            if (first) a.out.tile_col[e0 + at + __popcll(firsts & ((1ull << lane) - 1ull))] = t;
            if (a.ub) {
                // products per row: differences of the running sum at the ends of the rows' stretches in this wave
                const uint32_t inc = wave_inclusive_scan((uint32_t)len);
                const int r_next = __shfl_down(r, 1, 64), r_prev = __shfl_up(r, 1, 64);
                if (on && (lane == 63 || r_next != r)) atomicAdd(&s_ub[team][r], (unsigned long long)inc);
                if (on && lane > 0 && r_prev != r)
                    atomicAdd(&s_ub[team][r], (unsigned long long)0 - (unsigned long long)(inc - (uint32_t)len));
            }
        }
        const int e = wave_max((int)(range >> 16)), g = wave_max((int)(range & 0xFFFFu));
        if (lane == 0) {
            if constexpr (kTeam == 64) s_count[team] = listed;
            atomicMax(&s_range[0][team], (uint32_t)e);
            atomicMax(&s_range[1][team], (uint32_t)g);
        }
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (live) {
        if (tid == 0) {
            a.out.ntiles[I] = s_count[team];
            a.out.range[I] = s_range[0][team] << 16 | s_range[1][team];
        }
        if (a.ub && tid < T && I * T + tid < a.rows)
            a.ub[I * T + tid] = (int32_t)min(s_ub[team][tid], (unsigned long long)INT32_MAX);
        if (bad && a.validate) a.d_scalars[S_INVALID] = 1;
    }
}

struct PlanArgs {
    int64_t a_rows, a_tile_rows, b_tile_rows;
    const int32_t *a_start, *ub, *a_ntiles, *a_tile_col, *b_ntiles;
    const uint32_t *a_range, *b_range;
    int same;                            // A and B are one matrix
    int merge_lanes;                     // most entries of a row of A that is merged
    int windows;                         // of columns of C, for the heavy rows
    int32_t *heavy;                      // rows that are not merged
    int4 *tasks;                         // {row, index into heavy, first window, one past the last window}
    int64_t heavy_cap, task_cap;
    int64_t *d_scalars, *h_scalars_dev;
    int64_t publish_tag;                 // 0: the sizes stay on the device
    unsigned long long *partial;         // [kPlanBlocks][kPlanSums]
};

__device__ __forceinline__ bool merged_row(int32_t entries, int32_t products, int merge_lanes) {
    return entries <= merge_lanes && products <= kMergeProducts;
}

// Sixteen lanes per tile-row: its candidate pairs (sum of the tiles of B's tile-rows behind its tiles), then a lane per
// row: merged or heavy, and how many tasks a heavy row makes.
__global__ __launch_bounds__(256) void k_row_plan(const PlanArgs a) {
    __shared__ unsigned long long s_sum[kPlanSums];
    __shared__ unsigned long long s_max[kPlanSums];
    __shared__ int s_last;
    if (threadIdx.x < kPlanSums) s_sum[threadIdx.x] = s_max[threadIdx.x] = 0;
    __syncthreads();
    const int lane = lane_id(), r = threadIdx.x & 15;
    unsigned long long cand = 0, tiles_a = 0, tiles_b = 0, products = 0, merged = 0;
    uint32_t range_a = 0, range_b = 0;
    int longest = 0;                     // heavy row of A
    const int groups = (a.windows + kGroupWindows - 1) / kGroupWindows;
    unsigned long long *counters = reinterpret_cast<unsigned long long *>(a.d_scalars + S_ROW_LISTS);
    const int64_t step = (int64_t)gridDim.x * 16;
    const int64_t most = a.a_tile_rows > a.b_tile_rows ? a.a_tile_rows : a.b_tile_rows;
    for (int64_t base = (int64_t)blockIdx.x * 16; base < most; base += step) {
        const int64_t I = base + (threadIdx.x >> 4);
        if (r == 0 && I < a.b_tile_rows && !a.same) {
            tiles_b += (unsigned)a.b_ntiles[I];
            range_b = range_max(range_b, a.b_range[I]);
        }
        int tasks = 0;
        bool heavy = false;
        const int64_t row = I * T + r;
        if (I < a.a_tile_rows) {
            const int32_t e0 = a.a_start[I * T], n = a.a_ntiles[I];
            if (r == 0) {
                tiles_a += (unsigned)n;
                range_a = range_max(range_a, a.a_range[I]);
            }
            for (int32_t j = r; j < n; j += 16) {
                const int32_t K = a.a_tile_col[e0 + j];
                if (K < a.b_tile_rows) cand += (unsigned)a.b_ntiles[K];
            }
            if (row < a.a_rows) {
                const int32_t deg = a.a_start[row + 1] - a.a_start[row], ub = a.ub[row];
                products += (unsigned)ub;
                heavy = deg > 0 && !merged_row(deg, ub, a.merge_lanes) && ub > 0;
                merged += !heavy && ub > 0;
                if (heavy) {
                    tasks = min(max(ub / kTaskProducts, 1), groups);
                    longest = max(longest, deg);
                }
            }
        }
        const unsigned long long heavies = __ballot(heavy);
        if (heavies) {                   // (uniform in the wave) places in both lists from one atomic
            const uint32_t inc = wave_inclusive_scan((uint32_t)tasks);
            unsigned long long at = 0;
            if (lane == 63) at = atomicAdd(counters, ((unsigned long long)__popcll(heavies) << 36) | inc);
            at = __shfl(at, 63, 64);
            const int64_t h = (int64_t)(at >> 36) + __popcll(heavies & ((1ull << lane) - 1ull));
            const int64_t t0 = (int64_t)(at & ((1ull << 36) - 1ull)) + inc - tasks;
            if (heavy && h < a.heavy_cap) {
                a.heavy[h] = (int32_t)row;
                // (groups of windows, as even as they go)
                for (int t = 0; t < tasks; ++t)
                    if (t0 + t < a.task_cap)
                        a.tasks[t0 + t] = make_int4((int)row, (int)h, (int)((int64_t)groups * t / tasks) * kGroupWindows,
                                                    min((int)((int64_t)groups * (t + 1) / tasks) * kGroupWindows, a.windows));
            }
        }
    }
    auto add = [&](int slot, unsigned long long v) {
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (lane == 0 && v) atomicAdd(&s_sum[slot], v);
    };
    add(0, cand);
    add(1, tiles_a);
    add(2, tiles_b);
    add(3, products);
    add(4, merged);
    auto most_of = [&](int slot, int v) {
        v = wave_max(v);
        if (lane == 0 && v) atomicMax(&s_max[slot], (unsigned long long)v);
    };
    most_of(0, (int)(range_a >> 16));
    most_of(1, (int)(range_a & 0xFFFFu));
    most_of(2, (int)(range_b >> 16));
    most_of(3, (int)(range_b & 0xFFFFu));
    most_of(4, longest);
    __syncthreads();
    // (sums of counts stay below 2^48, and so does the word that carries the maxima)
    if (threadIdx.x == 0) {
        s_sum[5] = s_max[0] << 48 | s_max[1] << 32 | s_max[2] << 16 | s_max[3];
        s_sum[6] = s_max[4];
    }
    __syncthreads();
    if (threadIdx.x < kPlanSums)
        __hip_atomic_store(&a.partial[blockIdx.x * kPlanSums + threadIdx.x], s_sum[threadIdx.x], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = atomicAdd(reinterpret_cast<unsigned long long *>(a.d_scalars + S_ROW_DONE), 1ull) == gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    // the last block to finish adds up the partial sums and hands the sizes to the host
    if (threadIdx.x < kPlanSums) s_sum[threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x < kPlanSums) s_max[threadIdx.x] = 0;
    __syncthreads();
    for (unsigned i = threadIdx.x; i < gridDim.x * kPlanSums; i += 256) {
        const unsigned long long v = __hip_atomic_load(&a.partial[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned slot = i % kPlanSums;
        if (!v) continue;
        if (slot == 5)
            for (int q = 0; q < 4; ++q) atomicMax(&s_max[q], (v >> (48 - 16 * q)) & 0xFFFFull);
        else if (slot == 6) atomicMax(&s_max[4], v);
        else atomicAdd(&s_sum[slot], v);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.d_scalars[S_CANDIDATES] = (int64_t)s_sum[0];
        a.d_scalars[S_TILES_A] = (int64_t)s_sum[1];
        a.d_scalars[S_TILES_B] = (int64_t)(a.same ? s_sum[1] : s_sum[2]);
        a.d_scalars[S_ROW_PRODUCTS] = (int64_t)s_sum[3];
        a.d_scalars[S_ROW_MERGED] = (int64_t)s_sum[4];
        const int from = a.same ? 0 : 2;
        a.d_scalars[S_ROW_RANGE_A] = (int64_t)(s_max[0] << 16 | s_max[1]);
        a.d_scalars[S_ROW_RANGE_B] = (int64_t)(s_max[from] << 16 | s_max[from + 1]);
        a.d_scalars[S_ROW_LONGEST] = (int64_t)s_max[4];
        const unsigned long long lists = __hip_atomic_load(counters, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.d_scalars[S_ROW_HEAVY] = (int64_t)(lists >> 36);
        a.d_scalars[S_ROW_TASKS] = (int64_t)(lists & ((1ull << 36) - 1ull));
        a.d_scalars[S_ROW_LISTS] = 0;
        a.d_scalars[S_ROW_DONE] = 0;
    }
    if (a.publish_tag) publish_scalars(a.d_scalars, a.h_scalars_dev, a.publish_tag);
}

// ---- merged rows ------------------------------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ int lanes_min(int v) {
    if constexpr (G == 8) {
        v = min(v, TSP_DPP(v, v, 0xB1, 0xf, false));      // quad_perm [1,0,3,2]
        v = min(v, TSP_DPP(v, v, 0x4E, 0xf, false));      // quad_perm [2,3,0,1]
        v = min(v, TSP_DPP(v, v, 0x141, 0xf, false));     // row_half_mirror
        return v;
    } else {
        return group16_min(v);
    }
}
template <int G>
__device__ __forceinline__ float lanes_sum(float v) {     // the same tree, and so the same bits, in all lanes of the group
#define TSP_ADD_DPP(ctrl) v = v + __uint_as_float((uint32_t)TSP_DPP((int)__float_as_uint(v), (int)__float_as_uint(v), ctrl, 0xf, false))
    if constexpr (G == 8) {
        TSP_ADD_DPP(0xB1);
        TSP_ADD_DPP(0x4E);
        TSP_ADD_DPP(0x141);
    } else {
        TSP_ADD_DPP(0x128);
        TSP_ADD_DPP(0x124);
        TSP_ADD_DPP(0x122);
        TSP_ADD_DPP(0x121);
    }
#undef TSP_ADD_DPP
    return v;
}

struct MergeArgs {
    int64_t rows;
    const int32_t *a_start, *b_start, *ub;
    const int2 *a_rec, *b_rec;
    // sizing pass
    int32_t *row_nnz;
    uint32_t *group_len;                 // entries per 16 rows
    // multiplication pass
    const int64_t *c_row_ptr;
    int32_t *c_col;
    float *c_val;
    int stage;                           // entries of the output a wave keeps in LDS
    int64_t *d_scalars_to_clear;
};

// A group of G lanes per row of A, a lane per entry a_ik: every lane holds the next entry of its row of B, and a step
// takes the smallest column of the group and adds up the lanes that stand at it.  One entry of C per step, in column
// order; the next entry of every list is requested one step ahead.  The sizing pass counts the steps, the
// multiplication pass collects the entries of its wave's rows, which are neighbours in C, in LDS and writes them whole.
template <int G, bool kFill>
__global__ __launch_bounds__(256) void k_row_merge(const MergeArgs a) {
    constexpr int kRows = 64 / G;        // per wave
    extern __shared__ uint32_t lds_stage[];
    __shared__ uint32_t s_len[256 / G];
    const int lane = lane_id(), l = lane % G, wave = threadIdx.x >> 6;
    const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
    if constexpr (kFill)
        if (a.d_scalars_to_clear && blockIdx.x == 0 && threadIdx.x < kScalars) a.d_scalars_to_clear[threadIdx.x] = 0;
    int32_t p = 0, e = 0, deg = 0, ub = 0;
    float av = 0.f;
    bool merged = false;
    if (row < a.rows) {
        const int32_t s = a.a_start[row];
        deg = a.a_start[row + 1] - s;
        ub = a.ub[row];
        merged = ub > 0 && merged_row(deg, ub, G);
        if (merged && l < deg) {
            const int2 x = a.a_rec[s + l];
            p = a.b_start[x.x];
            e = a.b_start[x.x + 1];
            av = __uint_as_float((uint32_t)x.y);
        }
    }
    int2 head = make_int2(kNoCol, 0), next = head;
    if (p < e) head = a.b_rec[p];
    if (p + 1 < e) next = a.b_rec[p + 1];
    p += 2;
    if constexpr (!kFill) {
        int count = 0;
        while (true) {
            const int m = lanes_min<G>(head.x);
            const bool more = m != kNoCol;
            if (!__any(more)) break;
            count += more ? 1 : 0;
            if (more && head.x == m) {
                head.x = next.x;
                next.x = kNoCol;
                if (p < e) next.x = a.b_rec[p].x;
                ++p;
            }
        }
        // (rows of other kernels count as empty here)
        if (l == 0) {
            if (row < a.rows && (merged || ub == 0 || deg == 0)) a.row_nnz[row] = count;
            s_len[threadIdx.x / G] = (uint32_t)count;
        }
        __syncthreads();
        const int64_t g = (int64_t)blockIdx.x * (256 / G / T) + threadIdx.x;
        if (threadIdx.x < 256 / G / T && g * T < a.rows) {
            uint32_t sum = 0;
            for (int i = 0; i < T; ++i) sum += s_len[threadIdx.x * T + i];
            a.group_len[g] = sum;
        }
    } else {
        int64_t first = 0;
        int n = 0;
        if (merged) {
            first = a.c_row_ptr[row];
            n = (int)(a.c_row_ptr[row + 1] - first);
        }
        // where the row's entries lie among those of the wave
        int off[kRows + 1];
        off[0] = 0;
#pragma unroll
        for (int i = 0; i < kRows; ++i) off[i + 1] = off[i] + __builtin_amdgcn_readlane(n, i * G);
        const int total = off[kRows];
        const bool staged = total <= a.stage;
        int at = 0;
#pragma unroll
        for (int i = 0; i < kRows; ++i)
            if (lane / G == i) at = off[i];
        uint32_t *st_col = lds_stage + wave * 2 * a.stage, *st_val = st_col + a.stage;
        int done = 0;
        while (true) {
            const int m = lanes_min<G>(head.x);
            const bool more = m != kNoCol;
            if (!__any(more)) break;
            const bool mine = more && head.x == m;
            const float sum = lanes_sum<G>(mine ? av * __uint_as_float((uint32_t)head.y) : 0.f);
            if (l == 0 && more && done < n) {
                if (staged) {
                    st_col[at + done] = (uint32_t)m;
                    st_val[at + done] = __float_as_uint(sum);
                } else {
                    a.c_col[first + done] = m;
                    a.c_val[first + done] = sum;
                }
            }
            ++done;
            if (mine) {
                head = next;
                next.x = kNoCol;
                if (p < e) next = a.b_rec[p];
                ++p;
            }
        }
        if (!staged) return;
        wave_sync();
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            // rows that follow one another in C without a gap are written in one go
            const int64_t to = __shfl(first, i * G, 64);
            for (int j = off[i] + lane; j < off[i + 1]; j += 64) {
                a.c_col[to + (j - off[i])] = (int32_t)st_col[j];
                a.c_val[to + (j - off[i])] = __uint_as_float(st_val[j]);
            }
        }
    }
}

// ---- heavy rows -------------------------------------------------------------------------------------------------
// B for the heavy rows: 4 bytes per entry {low 16 bits of the column, fp16 value}, and where every row of B enters
// every window of columns; the columns once more by themselves.  L lanes per row.
struct PackArgs {
    int64_t rows;
    const int32_t *start;
    const int2 *rec;
    uint32_t *pack;
    int32_t *col;
    int32_t *table;                      // [rows][windows + 1], or null for one window
    int windows, shift;                  // a window is 1 << shift columns
};
template <int L>
__global__ __launch_bounds__(256) void k_heavy_pack(const PackArgs a) {
    const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / L;
    const int l = threadIdx.x % L;
    if (row >= a.rows) return;
    const int32_t s = a.start[row], e = max(s, a.start[row + 1]);
    int32_t *tab = a.table ? a.table + row * (a.windows + 1) : nullptr;
    for (int32_t k = s + l; k < e; k += L) {
        const int2 x = a.rec[k];
        const _Float16 v = (_Float16)__uint_as_float((uint32_t)x.y);
        a.col[k] = x.x;
        a.pack[k] = ((uint32_t)x.x & 0xFFFFu) | ((uint32_t)__builtin_bit_cast(uint16_t, v) << 16);
        if (tab) {
            const int before = k > s ? a.rec[k - 1].x >> a.shift : -1;
            for (int w = before + 1; w <= (x.x >> a.shift) && w <= a.windows; ++w) tab[w] = k;
        }
    }
    if (tab) {
        const int last = e > s ? min(a.rec[e - 1].x >> a.shift, a.windows - 1) : -1;
        for (int w = last + 1 + l; w <= a.windows; w += L) tab[w] = e;
    }
}

// The segments of B behind up to 64 entries of A, one per lane (first entry, length, value a_ik), as a stream of pieces of
// at most 64 entries, segment by segment: load(p) fetches entry p + lane of a piece, apply(x, a) takes what a lane below
// the piece's length got.  Eight pieces are requested while the eight before them are applied, across the ends of
// segments, so that a memory round trip is paid once per chunk and not per segment; everything that steers the stream
// is scalar.  load must be allowed to read up to 63 entries past a segment.
template <typename X, typename Load, typename Apply>
__device__ __forceinline__ void stream_segments(int p, int len, int av, Load load, Apply apply) {
    constexpr int kBatch = 8;
    const int lane = lane_id();
    const unsigned long long some = __ballot(len > 0);
    if (!some) return;
    const unsigned long long below = (1ull << lane) - 1ull;
    // the segments that hold something, in the order of their lanes
    const int to = (len > 0 ? __popcll(some & below) : __popcll(some) + __popcll(~some & below)) * 4;
    p = __builtin_amdgcn_ds_permute(to, p);
    av = __builtin_amdgcn_ds_permute(to, av);
    len = __builtin_amdgcn_ds_permute(to, max(len, 0));
    int left = (int)wave_sum((uint32_t)(len + 63) >> 6);
    int i = 0, sp = __builtin_amdgcn_readlane(p, 0), sl = __builtin_amdgcn_readlane(len, 0);
    struct Batch {
        X x[kBatch];
        int n[kBatch];
        int a[kBatch];
    };
    auto fetch = [&](Batch &b) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            b.x[u] = load(sp);
            b.n[u] = u < left ? sl : 0;
            b.a[u] = __builtin_amdgcn_readlane(av, i);
            // (both ways in full, so that they become selects and not branches)
            const int j = (i + 1) & 63;
            const int p_next = __builtin_amdgcn_readlane(p, j), l_next = __builtin_amdgcn_readlane(len, j);
            const int p_on = sp + 64, l_on = sl - 64;
            const bool more = sl > 64;
            i = more ? i : j;
            sp = more ? p_on : p_next;
            sl = more ? l_on : l_next;
        }
        left -= kBatch;
    };
    auto use = [&](const Batch &b) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (lane < b.n[u]) apply(b.x[u], __uint_as_float((uint32_t)b.a[u]));
    };
    Batch b0, b1;
    fetch(b0);
    // (the next batch is requested also when there is none, 8 loads of no use: behind a branch the waits could not tell
    // the two batches apart)
    while (true) {
        const bool more = left > 0;
        fetch(b1);
        use(b0);
        if (!more) break;
        const bool again = left > 0;
        fetch(b0);
        use(b1);
        if (!again) break;
    }
}

struct CountArgs {
    const int32_t *heavy;
    int64_t heavy_cap;
    const int64_t *d_scalars;
    const int32_t *a_start, *b_start, *ub;
    const int2 *a_rec;
    const int32_t *b_col;
    const int32_t *table;
    int32_t b_nnz;
    int windows;                         // of kWin columns each
    int span_windows;                    // windows whose bits the block's LDS holds
    int32_t *row_nnz;
    uint32_t *group_len;
    uint32_t *offset;                    // [heavy][windows] entries of the row before each window
};

// A block per heavy row sets one bit per product in LDS; OR is free of order, so the row may be spread over the block.
// Long segments of B: a wave takes 64 entries of A at a time and streams the segments behind them.  Short ones: the
// segments behind 512 entries of A are listed in LDS and groups of 8 or 16 lanes take one each.
template <int kWin>
__global__ __launch_bounds__(kHeavyThreads) void k_heavy_count(const CountArgs a) {
    extern __shared__ __align__(16) uint32_t bits[];
    __shared__ int2 s_seg[kHeavyThreads];
    __shared__ uint32_t s_cnt[64];
    __shared__ uint32_t s_run;
    constexpr int kWords = kWin / 32, kPerLane = kWords / 64;
    const int64_t h = blockIdx.x;
    if (h >= a.heavy_cap || h >= a.d_scalars[S_ROW_HEAVY]) return;
    const int32_t row = a.heavy[h];
    const int32_t s = a.a_start[row], e = a.a_start[row + 1];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int w = threadIdx.x; w < a.span_windows * kWords; w += kHeavyThreads) bits[w] = 0;
    if (threadIdx.x == 0) s_run = 0;
    const int mean = e > s ? a.ub[row] / (e - s) : 0;            // length of the rows of B behind this row
    for (int w0 = 0; w0 < a.windows; w0 += a.span_windows) {
        const int w1 = min(w0 + a.span_windows, a.windows);
        const int32_t c0 = w0 * kWin;
        const uint32_t limit = (uint32_t)(w1 - w0) * kWin;
        auto segment = [&](int32_t entry) {
            const int32_t c = a.a_rec[entry].x;
            if (a.windows <= a.span_windows) return make_int2(a.b_start[c], a.b_start[c + 1]);
            const int32_t *tab = a.table + (int64_t)c * (a.windows + 1);
            return make_int2(max(tab[w0], 0), min(tab[w1], a.b_nnz));
        };
        auto mark = [&](int32_t col) {
            const uint32_t x = (uint32_t)(col - c0);
            if (x < limit) atomicOr(&bits[x >> 5], 1u << (x & 31));
        };
        __syncthreads();
        if (mean > 16) {
            for (int32_t base = s + wave * 64; base < e; base += kHeavyThreads) {
                int2 seg = make_int2(0, 0);
                if (base + lane < e) seg = segment(base + lane);
                stream_segments<int32_t>(
                    seg.x, seg.y - seg.x, 0, [&](int p) { return (a.b_col + p)[(unsigned)lane]; },
                    [&](int32_t col, float) { mark(col); });
            }
        } else {
            const int sh = mean > 8 ? 4 : 3, lanes = 1 << sh, subs = kHeavyThreads >> sh;
            const int sub = threadIdx.x >> sh, j0 = threadIdx.x & (lanes - 1);
            for (int32_t base = s; base < e; base += kHeavyThreads) {
                const int n = min(e - base, kHeavyThreads);
                __syncthreads();
                if ((int)threadIdx.x < n) s_seg[threadIdx.x] = segment(base + threadIdx.x);
                __syncthreads();
                for (int i = sub; i < n; i += 4 * subs) {
                    int32_t p[4], q[4], c[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int2 seg = s_seg[min(i + u * subs, n - 1)];
                        p[u] = seg.x + j0;
                        q[u] = i + u * subs < n ? seg.y : 0;
                        c[u] = p[u] < q[u] ? a.b_col[p[u]] : -1;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (p[u] < q[u]) mark(c[u]);
                        for (p[u] += lanes; p[u] < q[u]; p[u] += lanes) mark(a.b_col[p[u]]);
                    }
                }
            }
        }
        __syncthreads();
        for (int w = wave; w < w1 - w0; w += kHeavyThreads / 64) {
            uint32_t n = 0;
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
                uint32_t *word = &bits[w * kWords + i * 64 + lane];
                n += __popc(*word);
                *word = 0;
            }
            n = wave_sum(n);
            if (lane == 0) s_cnt[w] = n;
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t n = lane < w1 - w0 ? s_cnt[lane] : 0;
            const uint32_t inc = wave_inclusive_scan(n), before = s_run;
            if (lane < w1 - w0) a.offset[h * a.windows + w0 + lane] = before + inc - n;
            if (lane == 63) s_run = before + inc;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.row_nnz[row] = (int32_t)s_run;
        atomicAdd(&a.group_len[row / T], s_run);
    }
}

struct FillArgs {
    const int4 *tasks;
    int64_t n_tasks;
    const int32_t *a_start, *b_start;
    const int2 *a_rec;
    const uint32_t *pack;
    const int32_t *table;
    int32_t b_nnz;
    int windows;
    const uint32_t *offset;
    const int64_t *c_row_ptr;
    int32_t *c_col;
    float *c_val;
    int window;                          // columns
    float a_scale, b_scale, c_scale;     // integers from the values, values from the integer sums
    int64_t *d_scalars_to_clear;
};

// A block per task: a row of C, kWin columns at a time (some of its windows).  Its waves deal the entries of the row of
// A among them, 64 apiece, and stream the segments of B behind them into a dense accumulator in LDS, with a bit per
// column; then every wave lists the entries of 2048 columns from the bits (or, where more than a quarter is there, walks
// the columns) and writes them 64 to a store.  The segments of the next step and the entries of the one after are
// requested ahead.
//
// The accumulator: LDS adds an fp32 number one lane after the other (193 cycles for a wave's 64 lanes, measured), an
// integer or an fp64 number all lanes at a time (5, 8 and 8 to 16 cycles for 32-bit and 64-bit integers and fp64).  So
// the sums are integers where they are exact in them, and fp64 otherwise; fp64 only with a block of one wave, which
// fixes the order of the additions.
constexpr int kFillList = 512;           // entries a wave lists at a time
template <typename Acc, int kWin, int kThreads>
__global__ __launch_bounds__(kThreads) void k_heavy_fill(const FillArgs a) {
    constexpr int kWaves = kThreads / 64;
    extern __shared__ __align__(16) unsigned char fill_lds[];
    const int columns = min(kWin, a.windows * a.window);       // of a step
    Acc *acc = reinterpret_cast<Acc *>(fill_lds);
    uint32_t *bits = reinterpret_cast<uint32_t *>(acc + columns);
    uint16_t *list = reinterpret_cast<uint16_t *>(bits + columns / 32) + (threadIdx.x >> 6) * kFillList;
    __shared__ int s_total[kWaves];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    auto sync = [] {
        if constexpr (kThreads == 64) wave_sync();
        else __syncthreads();
    };
    if (a.d_scalars_to_clear && blockIdx.x == 0 && threadIdx.x < kScalars) a.d_scalars_to_clear[threadIdx.x] = 0;
    const int64_t t = blockIdx.x;
    if (t >= a.n_tasks) return;
    const int4 task = a.tasks[t];
    const int32_t row = task.x, s = a.a_start[row], e = a.a_start[row + 1];
    const int64_t row_first = a.c_row_ptr[row], row_end = a.c_row_ptr[row + 1];
    const int chunks = (e - s + kThreads - 1) / kThreads;      // every wave takes its 64 entries of each
    if (chunks <= 0 || task.z >= task.w) return;
    for (int i = threadIdx.x; i < columns * (int)sizeof(Acc) / 16; i += kThreads)
        reinterpret_cast<uint4 *>(acc)[i] = make_uint4(0, 0, 0, 0);
    for (int i = threadIdx.x; i < columns / 32; i += kThreads) bits[i] = 0;
    // (requested without branches around the loads, which would wait for them: lanes past the end repeat the last entry)
    auto entry_at = [&](int chunk) { return s + chunk * kThreads + lane * kWaves + wave; };
    auto entry = [&](int chunk) { return a.a_rec[min(entry_at(chunk), e - 1)]; };
    const int steps = kWin / a.window;                         // windows per step
    const bool one = a.table == nullptr;
    auto segment = [&](int32_t c, int w) {
        const int32_t *from = one ? a.b_start + c : a.table + ((int64_t)c * (a.windows + 1) + w);
        return make_int2(from[0], from[one ? 1 : min(steps, a.windows - w)]);
    };
    const uint32_t *offset = a.offset + (int64_t)task.y * a.windows;
    int w = task.z, chunk = 0, ahead = chunks > 1 ? 1 : 0;
    int2 x0 = entry(0), seg0 = segment(x0.x, w), x1 = entry(ahead);
    int64_t first = row_first + offset[w];
    sync();
    while (true) {
        const bool step_ends = chunk == chunks - 1;
        const int2 seg1 = segment(x1.x, min(step_ends ? w + steps : w, a.windows - 1));
        ahead = ahead == chunks - 1 ? 0 : ahead + 1;
        const int2 x2 = entry(ahead);
        // (in bounds whatever an operand that was not validated holds)
        const int32_t p = max(seg0.x, 0), q = entry_at(chunk) < e ? min(seg0.y, a.b_nnz) : 0;
        const float scaled = __uint_as_float((uint32_t)x0.y) * a.a_scale;
        const int av = sizeof(Acc) == 8 && !std::is_floating_point<Acc>::value ? (int)scaled : (int)__float_as_uint(scaled);
        stream_segments<uint32_t>(
            p, q - p, av, [&](int p) { return (a.pack + p)[(unsigned)lane]; },
            [&](uint32_t x, float f) {
                const uint32_t c = x & (uint32_t)(kWin - 1);
                const float b = (float)__builtin_bit_cast(_Float16, (uint16_t)(x >> 16));
                if constexpr (std::is_floating_point<Acc>::value) unsafeAtomicAdd(&acc[c], (double)(f * b));
                else if constexpr (sizeof(Acc) == 4) atomicAdd(&acc[c], (int)(f * b));
                else
                    atomicAdd(reinterpret_cast<unsigned long long *>(&acc[c]),
                              (unsigned long long)((long long)(int)__float_as_uint(f) * (int)(b * a.b_scale)));
                atomicOr(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(bits) + ((c >> 3) & ~3u)), 1u << (c & 31));
            });
        if (step_ends) {
            const int w_next = min(w + steps, task.w);
            const int64_t last = w_next < a.windows ? row_first + offset[w_next] : row_end;
            sync();
            for (int part0 = 0; part0 < columns; part0 += kWaves * 2048) {
                const int part = part0 + wave * 2048;
                uint32_t word = part < columns ? bits[part / 32 + lane] : 0u;
                const uint32_t n = __popc(word), inc = wave_inclusive_scan(n);
                const int total = __builtin_amdgcn_readlane((int)inc, 63);
                int64_t at = first;
                if constexpr (kWaves > 1) {
                    if (lane == 0) s_total[wave] = total;
                    __syncthreads();
                    int before = 0, all = 0;
#pragma unroll
                    for (int v = 0; v < kWaves; ++v) {
                        before += v < wave ? s_total[v] : 0;
                        all += s_total[v];
                    }
                    at += before;
                    first += all;
                } else {
                    first += total;
                }
                auto emit = [&](int64_t to, int c, Acc v) {
                    if (to >= last) return;
                    a.c_col[to] = w * a.window + c;
                    if constexpr (std::is_floating_point<Acc>::value) a.c_val[to] = (float)v;
                    else a.c_val[to] = (float)v * a.c_scale;
                };
                if (total > 0) bits[part / 32 + lane] = 0;
                if (total > kFillList) {
                    const uint32_t before = inc - n;
                    for (int i = 0; i < 32; ++i) {                     // two words, 64 columns
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)word, 2 * i);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)word, 2 * i + 1);
                        const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)before, 2 * i);
                        const int c = part + i * 64 + lane;
                        if ((lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1u) {
                            const Acc v = acc[c];
                            acc[c] = Acc(0);
                            emit(at + from + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)), c, v);
                        }
                    }
                } else if (total > 0) {
                    uint16_t *to = list + (inc - n);
                    while (word) {
                        *to++ = (uint16_t)(part + lane * 32 + __ffs((int)word) - 1);
                        word &= word - 1;
                    }
                    wave_sync();
                    for (int i0 = 0; i0 < total; i0 += 128) {
                        int c[2];
                        Acc v[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) c[u] = list[min(i0 + u * 64 + lane, total - 1)];
#pragma unroll
                        for (int u = 0; u < 2; ++u) v[u] = acc[c[u]];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int i = i0 + u * 64 + lane;
                            if (i < total) {
                                acc[c[u]] = Acc(0);
                                emit(at + i, c[u], v[u]);
                            }
                        }
                    }
                    wave_sync();
                }
                if constexpr (kWaves > 1)
                    if (part0 + kWaves * 2048 < columns) __syncthreads();
            }
            first = last;
            w += steps;
            if (w >= task.w) break;
            sync();
            chunk = 0;
        } else {
            ++chunk;
        }
        x0 = x1;
        seg0 = seg1;
        x1 = x2;
    }
}

// ---- host ---------------------------------------------------------------------------------------------------------
namespace {

struct Workspace {                       // everything the path allocates, released together
    tsp_context *ctx;
    hipStream_t s;
    std::vector<void *> blocks;
    bool failed = false;
    template <typename Tp>
    Tp *get(size_t n) {
        Tp *p = ctx_alloc_n<Tp>(ctx, n, s);
        if (p) blocks.push_back(p);
        else failed = true;
        return p;
    }
    void keep(void *p) { blocks.erase(std::find(blocks.begin(), blocks.end(), p)); }
    ~Workspace() {
        for (void *p : blocks) ctx_free(ctx, p, s);
    }
};

template <typename RP, typename VT>
void launch_prepare(const PrepareArgs<RP, VT> &a, hipStream_t s) {
    const int64_t tile_rows = (a.rows + T - 1) / T;
    if (tile_rows == 0) return;
    // a wave per tile-row while a tile-row is a few dozen trips at most; longer ones get a block
    if (a.nnz <= 2048 * tile_rows && (size_t)a.bitmap_words * 16 <= 60 * 1024)
        hipLaunchKernelGGL((k_row_prepare<64, RP, VT>), dim3((unsigned)((tile_rows + 3) / 4)), dim3(256),
                           (size_t)a.bitmap_words * 16, s, a);
    else
        hipLaunchKernelGGL((k_row_prepare<256, RP, VT>), dim3((unsigned)tile_rows), dim3(256),
                           (size_t)a.bitmap_words * 4, s, a);
}

void prepare(tsp_context *ctx, const tsp_csr *M, const RowMatrix &out, int32_t *ub, const tsp_csr *B, hipStream_t s) {
    auto run = [&](auto rp, auto v) {
        using RP = decltype(rp);
        using VT = decltype(v);
        PrepareArgs<RP, VT> a{};
        a.row_ptr = static_cast<const RP *>(M->row_ptr);
        a.col = M->col_idx;
        a.val = static_cast<const VT *>(M->val);
        a.rows = M->rows;
        a.cols = M->cols;
        a.nnz = M->nnz;
        a.bitmap_words = (int)((M->cols + T * 32 - 1) / (T * 32));
        a.validate = ctx->validate;
        a.out = out;
        a.ub = ub;
        a.b_row_ptr = B->row_ptr;
        a.b_is_i64 = B->row_ptr_type == TSP_I64;
        a.b_rows = B->rows;
        a.b_nnz = B->nnz;
        a.d_scalars = ctx->d_scalars;
        launch_prepare(a, s);
    };
    const bool f16 = M->val_type == TSP_F16;
    if (M->row_ptr_type == TSP_I32) f16 ? run(int32_t{}, uint16_t{}) : run(int32_t{}, float{});
    else f16 ? run(int64_t{}, uint16_t{}) : run(int64_t{}, float{});
}

// Which accumulator is exact: the bits of the operands' values as integers (multiples of their common granularity), and
// of a sum of as many products as the longest heavy row of A has entries.
void launch_fill(FillArgs &f, const int64_t *h, hipStream_t s) {
    const int ra = (int)h[S_ROW_RANGE_A], rb = (int)h[S_ROW_RANGE_B];
    const int ea = (ra >> 16) - 256, ga = 256 - (ra & 0xFFFF), eb = (rb >> 16) - 256, gb = 256 - (rb & 0xFFFF);
    const bool finite = (ra >> 16) < 1023 && (rb >> 16) < 1023;
    int bits = ea - ga + eb - gb;
    for (int64_t n = 1; n < h[S_ROW_LONGEST]; n <<= 1) ++bits;
    const int columns = f.windows * f.window;
    auto launch = [&](auto kernel, int acc_bytes, int win, int threads) {
        const int step = std::min(columns, win);
        const size_t lds = (size_t)step * acc_bytes + step / 8 + (size_t)(threads / 64) * kFillList * 2;
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kernel, dim3((unsigned)f.n_tasks), dim3(threads), lds, s, f);
    };
    if (finite && ra && rb && bits <= 31) {
        f.a_scale = std::ldexp(1.0f, -(ga + gb));
        f.c_scale = std::ldexp(1.0f, ga + gb);
        launch(k_heavy_fill<int32_t, 16384, 512>, 4, 16384, 512);
    } else if (finite && ra && rb && bits <= 63 && ea - ga <= 31 && eb - gb <= 31) {
        f.a_scale = std::ldexp(1.0f, -ga);
        f.b_scale = std::ldexp(1.0f, -gb);
        f.c_scale = std::ldexp(1.0f, ga + gb);
        launch(k_heavy_fill<long long, 8192, 512>, 8, 8192, 512);
    } else {
        f.a_scale = 1.0f;
        launch(k_heavy_fill<double, 4096, 64>, 8, 4096, 64);
    }
}

}  // namespace

// The product A*B has so few intermediate products per candidate pair of tiles that the row kernels are faster.
static bool rows_preferred(int64_t products, int64_t candidates) { return products <= kRowPairProducts * candidates; }

int rowwise_spgemm(tsp_context *ctx, const tsp_csr *A, const tsp_csr *B, bool alias, tsp_csr *C, hipStream_t s,
                   bool *taken) {
    *taken = false;
    // Options that choose among the tile kernels, and shapes this path is not for: fewer rows than CUs (the sizing pass
    // has a block per heavy row), rows of more columns than the bitmaps of k_row_prepare hold (60 KB)
    if (!ctx->matrix_cores || ctx->numeric_run_len || ctx->work_order || ctx->strip_order || ctx->force_wide) return TSP_OK;
    int64_t most_cols = (int64_t)60 * 1024 * 8 * T;
    if (A->rows < 256 || A->rows > (1 << 27) || A->nnz == 0 || B->nnz == 0 || A->cols > most_cols || B->cols > most_cols) return TSP_OK;
    RowHint &hint = ctx->row_hint;
    const int64_t sizes[6] = {A->rows, A->nnz, B->rows, B->nnz, B->cols, alias};
    const bool known = std::equal(sizes, sizes + 6, hint.sizes);
    if (known && hint.tiles) return TSP_OK;

    const int64_t a_ntr = (A->rows + T - 1) / T, b_ntr = (B->rows + T - 1) / T;
    const int merge_lanes = A->nnz <= 8 * A->rows ? 8 : 16;
    const int shift = B->cols <= 2048 ? 11 : 12;
    const int windows = (int)((B->cols + (1 << shift) - 1) >> shift);
    const bool table_fits = windows == 1 || (B->rows * (windows + 1) * 4 <= (int64_t)4 << 30);

    Workspace ws{ctx, s, {}};
    RowMatrix ma, mb;
    auto take = [&](RowMatrix &m, const tsp_csr *M, int64_t ntr) {
        m.start = ws.get<int32_t>((size_t)M->rows + 1);
        m.rec = ws.get<int2>((size_t)M->nnz);
        m.ntiles = ws.get<int32_t>((size_t)ntr);
        m.tile_col = ws.get<int32_t>((size_t)M->nnz);
        m.range = ws.get<uint32_t>((size_t)ntr);
    };
    take(ma, A, a_ntr);
    if (alias) mb = ma;
    else take(mb, B, b_ntr);
    int32_t *ub = ws.get<int32_t>((size_t)A->rows);
    unsigned long long *partial = ws.get<unsigned long long>((size_t)kPlanBlocks * kPlanSums);
    int64_t heavy_cap = known ? hint.heavy : A->rows, task_cap = known ? hint.tasks : 0;
    if (!known) {
        // (tasks: one per heavy row and one more per kTaskProducts products, at most one per window; the products are not
        // known yet, so a second plan run follows in the rare case that this guess is too small)
        task_cap = std::min<int64_t>(A->rows * (int64_t)windows, 2 * A->rows + 4096);
    }
    int32_t *heavy = ws.get<int32_t>((size_t)std::max<int64_t>(heavy_cap, 1));
    int4 *tasks = ws.get<int4>((size_t)std::max<int64_t>(task_cap, 1));
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;

    phase_begin(ctx, TSP_PHASE_CONVERT, s);
    {
        KernelTimer kt(ctx, TSP_KERNEL_CONVERT, s);
        prepare(ctx, A, ma, ub, B, s);
        if (!alias) prepare(ctx, B, mb, nullptr, B, s);
    }
    phase_end(ctx, TSP_PHASE_CONVERT, s);
    TSP_HIP_CHECK(ctx, hipGetLastError());

    phase_begin(ctx, TSP_PHASE_SYMBOLIC, s);
    auto plan = [&](bool publish) {
        PlanArgs a{};
        a.a_rows = A->rows;
        a.a_tile_rows = a_ntr;
        a.b_tile_rows = b_ntr;
        a.a_start = ma.start;
        a.ub = ub;
        a.a_ntiles = ma.ntiles;
        a.a_tile_col = ma.tile_col;
        a.b_ntiles = mb.ntiles;
        a.a_range = ma.range;
        a.b_range = mb.range;
        a.same = alias;
        a.merge_lanes = merge_lanes;
        a.windows = windows;
        a.heavy = heavy;
        a.tasks = tasks;
        a.heavy_cap = heavy_cap;
        a.task_cap = task_cap;
        a.d_scalars = ctx->d_scalars;
        a.h_scalars_dev = ctx->h_scalars_dev;
        a.publish_tag = publish ? ++ctx->publish_tag : 0;
        a.partial = partial;
        const int64_t blocks = std::min<int64_t>(kPlanBlocks, (std::max(a_ntr, b_ntr) + 15) / 16);
        KernelTimer kt(ctx, TSP_KERNEL_SCAN_SYM, s);
        hipLaunchKernelGGL(k_row_plan, dim3((unsigned)blocks), dim3(256), 0, s, a);
    };
    plan(!known);
    TSP_HIP_CHECK(ctx, hipGetLastError());
    int64_t n_heavy = heavy_cap, n_tasks = task_cap;
    bool any_merged = !known || hint.merged;
    auto sizes_known = [&]() {               // the host has the numbers of k_row_plan
        const int64_t *h = ctx->h_scalars;
        if (h[S_INVALID]) return (int)TSP_ERR_NOT_CANONICAL;
        if (h[S_INTERNAL]) return (int)TSP_ERR_HIP;
        n_heavy = h[S_ROW_HEAVY];
        n_tasks = h[S_ROW_TASKS];
        any_merged = h[S_ROW_MERGED] > 0;
        std::copy(sizes, sizes + 6, hint.sizes);
        hint.tiles = !rows_preferred(h[S_ROW_PRODUCTS], h[S_CANDIDATES]) || (n_heavy > 0 && !table_fits) ||
                     n_tasks >= INT32_MAX;
        hint.heavy = n_heavy;
        hint.tasks = n_tasks;
        hint.merged = any_merged;
        return (int)TSP_OK;
    };
    if (!known) {
        int rc = wait_published_scalars(ctx, ctx->publish_tag, s);
        if (!rc) rc = sizes_known();
        if (rc) return rc;
        if (hint.tiles) return TSP_OK;       // (the tile kernels start over; the scalars they use are cleared for them)
    }
    *taken = true;

    int64_t *row_ptr = ws.get<int64_t>((size_t)A->rows + 1);
    int32_t *row_nnz = ws.get<int32_t>((size_t)A->rows + 1);
    uint32_t *group_len = ws.get<uint32_t>((size_t)a_ntr + 4);
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;
    uint32_t *pack = nullptr, *offset = nullptr;
    int32_t *table = nullptr, *heavy_col = nullptr;
    auto size_rows = [&]() {
        if (n_tasks > task_cap || n_heavy > heavy_cap) {
            // the lists did not fit: make them again, as large as they have to be
            heavy_cap = n_heavy;
            task_cap = n_tasks;
            heavy = ws.get<int32_t>((size_t)heavy_cap);
            tasks = ws.get<int4>((size_t)task_cap);
            if (ws.failed) return (int)TSP_ERR_ALLOC_FAILED;
            plan(false);
        }
        if (n_heavy > 0) {
            if (!pack) {
                pack = ws.get<uint32_t>((size_t)B->nnz + 64);     // (a piece is read whole)
                heavy_col = ws.get<int32_t>((size_t)B->nnz + 64);
                if (windows > 1) table = ws.get<int32_t>((size_t)B->rows * (windows + 1));
            }
            offset = ws.get<uint32_t>((size_t)n_heavy * windows);
            if (ws.failed) return (int)TSP_ERR_ALLOC_FAILED;
        }
        KernelTimer kt(ctx, TSP_KERNEL_SYM_COUNT, s);
        MergeArgs m{};
        m.rows = A->rows;
        m.a_start = ma.start;
        m.b_start = mb.start;
        m.ub = ub;
        m.a_rec = ma.rec;
        m.b_rec = mb.rec;
        m.row_nnz = row_nnz;
        m.group_len = group_len;
        auto merge = merge_lanes == 8 ? k_row_merge<8, false> : k_row_merge<16, false>;
        hipLaunchKernelGGL(merge,
                           dim3((unsigned)((A->rows * merge_lanes + 255) / 256)), dim3(256), 0, s, m);
        if (n_heavy > 0) {
            PackArgs p{B->rows, mb.start, mb.rec, pack, heavy_col, table, windows, shift};
            if (B->nnz > 16 * B->rows)
                hipLaunchKernelGGL(k_heavy_pack<64>, dim3((unsigned)((B->rows * 64 + 255) / 256)), dim3(256), 0, s, p);
            else
                hipLaunchKernelGGL(k_heavy_pack<16>, dim3((unsigned)((B->rows * 16 + 255) / 256)), dim3(256), 0, s, p);
            CountArgs c{};
            c.heavy = heavy;
            c.heavy_cap = n_heavy;
            c.d_scalars = ctx->d_scalars;
            c.a_start = ma.start;
            c.b_start = mb.start;
            c.ub = ub;
            c.a_rec = ma.rec;
            c.b_col = heavy_col;
            c.table = table;
            c.b_nnz = (int32_t)B->nnz;
            c.windows = windows;
            c.span_windows = std::min(windows, kSpanWindows);
            c.row_nnz = row_nnz;
            c.group_len = group_len;
            c.offset = offset;
            const size_t lds = (size_t)c.span_windows << (shift - 3);
            auto kernel = shift == 11 ? k_heavy_count<2048> : k_heavy_count<4096>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)n_heavy), dim3(kHeavyThreads), lds, s, c);
        }
        return (int)TSP_OK;
    };
    auto offsets = [&]() {                   // row_ptr of C, nnz(C) to the host: the wait that sizes C
        bool published = false;
        {
            KernelTimer kt(ctx, TSP_KERNEL_SCAN_ROWS, s);
            published = row_ptr_in_one_launch(ctx, row_nnz, A->rows, group_len, row_ptr, s);
            if (!published) {
                int64_t *tmp = ws.get<int64_t>(scan_tmp_entries(A->rows));
                if (!tmp) return (int)TSP_ERR_ALLOC_FAILED;
                int rc = scan_exclusive_i32_to_i64(ctx, row_nnz, row_ptr, A->rows, ctx->d_scalars + S_C_NNZ, nullptr, tmp, s);
                if (rc) return rc;
            }
        }
        TSP_HIP_CHECK(ctx, hipGetLastError());
        return published ? wait_published_scalars(ctx, ctx->publish_tag, s) : read_scalars(ctx, s);
    };
    int rc = size_rows();
    if (rc) return rc;
    phase_end(ctx, TSP_PHASE_SYMBOLIC, s);
    phase_begin(ctx, TSP_PHASE_COUNT, s);
    rc = offsets();
    if (rc) return rc;
    if (known) {
        const int64_t had_heavy = n_heavy, had_tasks = n_tasks;
        rc = sizes_known();
        if (rc) return rc;
        if (n_heavy > had_heavy || n_tasks > had_tasks) {       // another matrix of the same sizes, with more work in it
            rc = size_rows();
            if (!rc) rc = offsets();
            if (rc) return rc;
        }
    }
    phase_end(ctx, TSP_PHASE_COUNT, s);
    const int64_t nnz = ctx->h_scalars[S_C_NNZ];
    int32_t *col = ws.get<int32_t>((size_t)nnz);
    float *val = ws.get<float>((size_t)nnz);
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;

    phase_begin(ctx, TSP_PHASE_NUMERIC, s);
    {
        KernelTimer kt(ctx, TSP_KERNEL_NUMERIC, s);
        // (nothing reads the scalar block any more: the last kernel clears it for the next call)
        int64_t *clear = ctx->compact ? nullptr : ctx->d_scalars;
        bool cleared = false;
        if (any_merged && nnz > 0) {
            MergeArgs m{};
            m.rows = A->rows;
            m.a_start = ma.start;
            m.b_start = mb.start;
            m.ub = ub;
            m.a_rec = ma.rec;
            m.b_rec = mb.rec;
            m.c_row_ptr = row_ptr;
            m.c_col = col;
            m.c_val = val;
            // entries of C a wave collects: twice the mean of its rows, at most 8 KB
            const int64_t mean = nnz * (64 / merge_lanes) / A->rows;
            m.stage = 128;
            while (m.stage < 1024 && m.stage < 2 * mean) m.stage <<= 1;
            m.d_scalars_to_clear = n_tasks > 0 ? nullptr : clear;
            cleared = m.d_scalars_to_clear != nullptr;
            auto merge = merge_lanes == 8 ? k_row_merge<8, true> : k_row_merge<16, true>;
            hipLaunchKernelGGL(merge,
                               dim3((unsigned)((A->rows * merge_lanes + 255) / 256)), dim3(256), (size_t)m.stage * 32, s, m);
        }
        if (n_tasks > 0) {
            FillArgs f{};
            f.tasks = tasks;
            f.n_tasks = n_tasks;
            f.a_start = ma.start;
            f.b_start = mb.start;
            f.a_rec = ma.rec;
            f.pack = pack;
            f.table = table;
            f.b_nnz = (int32_t)B->nnz;
            f.windows = windows;
            f.offset = offset;
            f.c_row_ptr = row_ptr;
            f.c_col = col;
            f.c_val = val;
            f.d_scalars_to_clear = clear;
            cleared = clear != nullptr;
            f.window = 1 << shift;
            launch_fill(f, ctx->h_scalars, s);
        }
        TSP_HIP_CHECK(ctx, hipGetLastError());
        ctx->scalars_clean = cleared;
    }
    phase_end(ctx, TSP_PHASE_NUMERIC, s);
    const int64_t *h = ctx->h_scalars;
    ctx->stats.a_tiles = h[S_TILES_A];
    ctx->stats.b_tiles = h[S_TILES_B];
    ctx->stats.candidate_pairs = h[S_CANDIDATES];
    ctx->stats.pairs = 0;                    // no task list and no output tiles on this path
    ctx->stats.c_tiles = 0;
    ctx->stats.c_nnz = nnz;
    fill_selection_criteria(ctx, A->rows, A->nnz, h[S_TILES_A]);
    ws.keep(row_ptr);
    ws.keep(col);
    ws.keep(val);
    C->rows = A->rows;
    C->cols = B->cols;
    C->nnz = nnz;
    C->row_ptr = row_ptr;
    C->col_idx = col;
    C->val = val;
    C->row_ptr_type = TSP_I64;
    C->val_type = TSP_F32;
    return TSP_OK;
}

}  // namespace tsp
