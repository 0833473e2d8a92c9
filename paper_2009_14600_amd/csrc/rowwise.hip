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
//   k_heavy_fill    a wave per row and window of columns, a dense fp32 accumulator in LDS
//
// Every sum of C is formed in one wave in a fixed order (the entries of the row of A ascending; in a merge step the
// lanes of the group as a tree), so runs are bit-identical.  Products of fp16 numbers are exact in fp32 and are
// accumulated in fp32, as on the matrix cores.
#include "common.hpp"

#include <algorithm>

namespace tsp {

constexpr int kMergeProducts = 256;      // a merged row has at most this many intermediate products
constexpr int kPlanBlocks = 128;         // blocks of k_row_plan
constexpr int kPlanSums = 8;
constexpr int kHeavySpan = 48 * 8192;    // columns whose bits fit the LDS of a block of k_heavy_count (48 KB)
constexpr int kHeavyThreads = 256;
constexpr int32_t kNoCol = 0x7FFFFFFF;
// Intermediate products behind one task of k_heavy_fill (a row, or some of its windows)
constexpr int kTaskProducts = 16384;
constexpr int64_t kRowPairProducts = 64; // products per candidate pair of tiles up to which the rows are the better way

struct RowMatrix {                       // an operand in the form the row kernels read
    int32_t *start = nullptr;            // int32[rows + 1], clamped to [0, nnz]
    int2 *rec = nullptr;                 // per entry {column (clamped), value rounded to fp16, as fp32 bits}
    int32_t *ntiles = nullptr;           // tiles of every tile-row
    int32_t *tile_col = nullptr;         // their columns, at the position of the tile-row's first entry; any order
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
        if (tid == 0) s_count[team] = 0;
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (live) {
        const int32_t e0 = s_ptr[team][0], e1 = s_ptr[team][T];
        int32_t listed = 0;
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
        if constexpr (kTeam == 64)
            if (tid == 0) s_count[team] = listed;
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (live) {
        if (tid == 0) a.out.ntiles[I] = s_count[team];
        if (a.ub && tid < T && I * T + tid < a.rows)
            a.ub[I * T + tid] = (int32_t)min(s_ub[team][tid], (unsigned long long)INT32_MAX);
        if (bad && a.validate) a.d_scalars[S_INVALID] = 1;
    }
}

struct PlanArgs {
    int64_t a_rows, a_tile_rows, b_tile_rows;
    const int32_t *a_start, *ub, *a_ntiles, *a_tile_col, *b_ntiles;
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
    __shared__ int s_last;
    if (threadIdx.x < kPlanSums) s_sum[threadIdx.x] = 0;
    __syncthreads();
    const int lane = lane_id(), r = threadIdx.x & 15;
    unsigned long long cand = 0, tiles_a = 0, tiles_b = 0, products = 0, merged = 0;
    unsigned long long *counters = reinterpret_cast<unsigned long long *>(a.d_scalars + S_ROW_LISTS);
    const int64_t step = (int64_t)gridDim.x * 16;
    const int64_t most = a.a_tile_rows > a.b_tile_rows ? a.a_tile_rows : a.b_tile_rows;
    for (int64_t base = (int64_t)blockIdx.x * 16; base < most; base += step) {
        const int64_t I = base + (threadIdx.x >> 4);
        if (r == 0 && I < a.b_tile_rows && !a.same) tiles_b += (unsigned)a.b_ntiles[I];
        int tasks = 0;
        bool heavy = false;
        const int64_t row = I * T + r;
        if (I < a.a_tile_rows) {
            const int32_t e0 = a.a_start[I * T], n = a.a_ntiles[I];
            if (r == 0) tiles_a += (unsigned)n;
            for (int32_t j = r; j < n; j += 16) {
                const int32_t K = a.a_tile_col[e0 + j];
                if (K < a.b_tile_rows) cand += (unsigned)a.b_ntiles[K];
            }
            if (row < a.a_rows) {
                const int32_t deg = a.a_start[row + 1] - a.a_start[row], ub = a.ub[row];
                products += (unsigned)ub;
                heavy = deg > 0 && !merged_row(deg, ub, a.merge_lanes) && ub > 0;
                merged += !heavy && ub > 0;
                if (heavy) tasks = min(max(ub / kTaskProducts, 1), a.windows);
            }
        }
        const unsigned long long heavies = __ballot(heavy);
        if (heavies) {                   // (uniform in the wave) places in both lists from one atomic
            if (tasks) tasks = (a.windows + (a.windows + tasks - 1) / tasks - 1) / ((a.windows + tasks - 1) / tasks);
            const uint32_t inc = wave_inclusive_scan((uint32_t)tasks);
            unsigned long long at = 0;
            if (lane == 63) at = atomicAdd(counters, ((unsigned long long)__popcll(heavies) << 36) | inc);
            at = __shfl(at, 63, 64);
            const int64_t h = (int64_t)(at >> 36) + __popcll(heavies & ((1ull << lane) - 1ull));
            const int64_t t0 = (int64_t)(at & ((1ull << 36) - 1ull)) + inc - tasks;
            if (heavy && h < a.heavy_cap) {
                a.heavy[h] = (int32_t)row;
                const int per = (a.windows + tasks - 1) / tasks;
                for (int t = 0; t < tasks; ++t)
                    if (t0 + t < a.task_cap)
                        a.tasks[t0 + t] = make_int4((int)row, (int)h, t * per, min((t + 1) * per, a.windows));
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
    for (unsigned i = threadIdx.x; i < gridDim.x * kPlanSums; i += 256) {
        const unsigned long long v = __hip_atomic_load(&a.partial[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v) atomicAdd(&s_sum[i % kPlanSums], v);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.d_scalars[S_CANDIDATES] = (int64_t)s_sum[0];
        a.d_scalars[S_TILES_A] = (int64_t)s_sum[1];
        a.d_scalars[S_TILES_B] = (int64_t)(a.same ? s_sum[1] : s_sum[2]);
        a.d_scalars[S_ROW_PRODUCTS] = (int64_t)s_sum[3];
        a.d_scalars[S_ROW_MERGED] = (int64_t)s_sum[4];
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
// every window of columns.  Sixteen lanes per row.
struct PackArgs {
    int64_t rows;
    const int32_t *start;
    const int2 *rec;
    uint32_t *pack;
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

struct CountArgs {
    const int32_t *heavy;
    int64_t heavy_cap;
    const int64_t *d_scalars;
    const int32_t *a_start, *b_start, *ub;
    const int2 *a_rec, *b_rec;
    const int32_t *table;
    int32_t b_nnz;
    int windows;                         // of kWin columns each
    int span_windows;                    // windows whose bits the block's LDS holds
    int32_t *row_nnz;
    uint32_t *group_len;
    uint32_t *offset;                    // [heavy][windows] entries of the row before each window
};

// A block per heavy row: the segments of B behind 256 entries of A at a time are listed in LDS, groups of lanes walk
// them and set one bit per product.  OR is free of order, so the row may be spread over the whole block.
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
    // lanes per segment, from the mean length of the rows of B behind this row
    const int mean = e > s ? a.ub[row] / (e - s) : 0;
    const int sh = mean > 32 ? 6 : mean > 16 ? 5 : mean > 8 ? 4 : 3;
    const int lanes = 1 << sh, sub = threadIdx.x >> sh, j0 = threadIdx.x & (lanes - 1), subs = kHeavyThreads >> sh;
    for (int w0 = 0; w0 < a.windows; w0 += a.span_windows) {
        const int w1 = min(w0 + a.span_windows, a.windows);
        const int32_t c0 = w0 * kWin;
        const uint32_t limit = (uint32_t)(w1 - w0) * kWin;
        for (int32_t base = s; base < e; base += kHeavyThreads) {
            const int n = min(e - base, kHeavyThreads);
            __syncthreads();
            if ((int)threadIdx.x < n) {
                const int32_t c = a.a_rec[base + threadIdx.x].x;
                int2 seg;
                if (a.windows <= a.span_windows) seg = make_int2(a.b_start[c], a.b_start[c + 1]);
                else seg = make_int2(max(a.table[(int64_t)c * (a.windows + 1) + w0], 0),
                                     min(a.table[(int64_t)c * (a.windows + 1) + w1], a.b_nnz));
                s_seg[threadIdx.x] = seg;
            }
            __syncthreads();
            auto mark = [&](int32_t col) {
                const uint32_t x = (uint32_t)(col - c0);
                if (x < limit) atomicOr(&bits[x >> 5], 1u << (x & 31));
            };
            for (int i = sub; i < n; i += 4 * subs) {
                int32_t p[4], q[4], c[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int2 seg = s_seg[min(i + u * subs, n - 1)];
                    p[u] = seg.x + j0;
                    q[u] = i + u * subs < n ? seg.y : 0;
                    c[u] = p[u] < q[u] ? a.b_rec[p[u]].x : -1;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (p[u] < q[u]) mark(c[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    for (p[u] += lanes; p[u] < q[u]; p[u] += 4 * lanes) {
                        int32_t d[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) d[v] = p[u] + v * lanes < q[u] ? a.b_rec[p[u] + v * lanes].x : -1;
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (p[u] + v * lanes < q[u]) mark(d[v]);
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
    int64_t *d_scalars_to_clear;
};

// A wave per task: a row of C, window by window of kWin columns.  The wave adds the products into a dense accumulator
// in LDS (its own: no other wave adds to it, so the order of the sums is fixed) and sets a bit per column; the entries
// are then listed from the bits, a word per lane and 2048 columns at a time, and written 64 to a store.
template <int kWin>
__global__ __launch_bounds__(64) void k_heavy_fill(const FillArgs a) {
    __shared__ float acc[kWin];
    __shared__ uint32_t bits[kWin / 32];
    __shared__ uint16_t list[2048];
    const int lane = threadIdx.x;
    if (a.d_scalars_to_clear && blockIdx.x == 0 && threadIdx.x < kScalars) a.d_scalars_to_clear[threadIdx.x] = 0;
    const int64_t t = blockIdx.x;
    if (t >= a.n_tasks) return;
    const int4 task = a.tasks[t];
    const int32_t row = task.x, s = a.a_start[row], e = a.a_start[row + 1];
    const int64_t row_first = a.c_row_ptr[row], row_end = a.c_row_ptr[row + 1];
    for (int i = lane; i < kWin; i += 64) acc[i] = 0.f;
    for (int i = lane; i < kWin / 32; i += 64) bits[i] = 0;
    wave_sync();
    for (int w = task.z; w < task.w; ++w) {
        const int64_t first = row_first + a.offset[(int64_t)task.y * a.windows + w];
        const int64_t last = w + 1 < a.windows ? row_first + a.offset[(int64_t)task.y * a.windows + w + 1] : row_end;
        if (first >= last) continue;
        for (int32_t base = s; base < e; base += 64) {
            int32_t p = 0, q = 0, av = 0;
            if (base + lane < e) {
                const int2 x = a.a_rec[base + lane];
                av = x.y;
                if (a.table) {
                    const int32_t *tab = a.table + (int64_t)x.x * (a.windows + 1) + w;
                    p = max(tab[0], 0);              // (in bounds whatever an operand that was not validated holds)
                    q = min(tab[1], a.b_nnz);
                } else {
                    p = a.b_start[x.x];
                    q = a.b_start[x.x + 1];
                }
            }
            unsigned long long left = __ballot(p < q);
            auto add = [&](uint32_t x, float f) {
                const uint32_t c = x & (kWin - 1);
                const float b = (float)__builtin_bit_cast(_Float16, (uint16_t)(x >> 16));
                unsafeAtomicAdd(&acc[c], f * b);
                atomicOr(&bits[c >> 5], 1u << (c & 31));
            };
            while (left) {
                constexpr int kBatch = 8;
                int32_t pu[kBatch], qu[kBatch];
                float au[kBatch];
                uint32_t x[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int src = left ? __ffsll((long long)left) - 1 : 0;
                    pu[u] = __builtin_amdgcn_readlane(p, src);
                    qu[u] = left ? __builtin_amdgcn_readlane(q, src) : 0;
                    au[u] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane(av, src));
                    left &= left - 1;
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) x[u] = pu[u] + lane < qu[u] ? a.pack[pu[u] + lane] : 0u;
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (pu[u] + lane < qu[u]) add(x[u], au[u]);
                    for (int32_t k = pu[u] + 64; k < qu[u]; k += 256) {
                        uint32_t y[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) y[v] = k + 64 * v + lane < qu[u] ? a.pack[k + 64 * v + lane] : 0u;
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (k + 64 * v + lane < qu[u]) add(y[v], au[u]);
                    }
                }
            }
        }
        wave_sync();
        int64_t at = first;
        for (int part = 0; part < kWin / 2048; ++part) {
            uint32_t word = bits[part * 64 + lane];
            const uint32_t n = __popc(word), inc = wave_inclusive_scan(n);
            const int total = __builtin_amdgcn_readlane((int)inc, 63);
            if (!total) continue;
            bits[part * 64 + lane] = 0;
            uint32_t to = inc - n;
            while (word) {
                const int b = __ffs((int)word) - 1;
                word &= word - 1;
                list[to++] = (uint16_t)(part * 2048 + lane * 32 + b);
            }
            wave_sync();
            for (int i = lane; i < total && at + i < last; i += 64) {
                const int c = list[i];
                a.c_col[at + i] = w * kWin + c;
                a.c_val[at + i] = acc[c];
                acc[c] = 0.f;
            }
            at += total;
            wave_sync();
        }
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
    // windows of columns of the heavy rows: one small one for a narrow C, else 8192 columns
    const int shift = B->cols <= 2048 ? 11 : B->cols <= 4096 ? 12 : 13;
    const int windows = (int)((B->cols + (1 << shift) - 1) >> shift);
    const bool table_fits = windows == 1 || (B->rows * (windows + 1) * 4 <= (int64_t)4 << 30);

    Workspace ws{ctx, s, {}};
    RowMatrix ma, mb;
    auto take = [&](RowMatrix &m, const tsp_csr *M, int64_t ntr) {
        m.start = ws.get<int32_t>((size_t)M->rows + 1);
        m.rec = ws.get<int2>((size_t)M->nnz);
        m.ntiles = ws.get<int32_t>((size_t)ntr);
        m.tile_col = ws.get<int32_t>((size_t)M->nnz);
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
    int32_t *table = nullptr;
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
                pack = ws.get<uint32_t>((size_t)B->nnz);
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
            PackArgs p{B->rows, mb.start, mb.rec, pack, table, windows, shift};
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
            c.b_rec = mb.rec;
            c.table = table;
            c.b_nnz = (int32_t)B->nnz;
            c.windows = windows;
            c.span_windows = (int)std::min<int64_t>(windows, kHeavySpan >> shift);
            c.row_nnz = row_nnz;
            c.group_len = group_len;
            c.offset = offset;
            const size_t lds = (size_t)c.span_windows << (shift - 3);
            auto kernel = shift == 11 ? k_heavy_count<2048> : shift == 12 ? k_heavy_count<4096> : k_heavy_count<8192>;
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
            auto kernel = shift == 11 ? k_heavy_fill<2048> : shift == 12 ? k_heavy_fill<4096> : k_heavy_fill<8192>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)n_tasks), dim3(64), 0, s, f);
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
