// C = A*B row by row (Gustavson's order), for operands whose 16x16 tiles hold too little for block products: a
// (A tile, B tile) pair of a graph or of a mesh with one unknown per node multiplies a handful of entries, and the
// task list, the counting pass and the block products all cost by the pair.  Here everything costs by the
// intermediate product a_ik * b_kj:
//
//   k_row_sample    operands of sizes not seen before: a look at some of their tile-rows, whether they are clearly for tiles
//   k_row_prepare   one pass over an operand: validation, entries as {column, value} records, tiles per tile-row,
//                   and for A the number of intermediate products of every row and the lists of work
//   k_row_finish    row_ptr of C; candidate tile pairs (the measure by which tsp_spgemm chooses this path) and other sums
//   k_row_small     rows with few, short rows of B behind them: products sorted in registers; k_small_copy puts them in place,
//                   or k_small_finish, which makes row_ptr as well, where no other rows are expected
//   k_row_given     where the last product of these sizes had no other rows: k_row_prepare's validation and tiles, and k_row_small
//                   straight from the operands, at once; k_given_finish makes row_ptr and puts the entries in place
//   k_heavy_pack    B for the other rows: words of 16 columns, entries of 4 bytes
//   k_heavy_count   their sizes: a block per row, one bit per column of C in LDS
//   k_heavy_fill    a block per row and some windows of columns, an accumulator in LDS for some thousand entries at a time
//
// A product that is repeated on a handle has the same bits every time.  Products of fp16 numbers are exact in fp32.  An entry of a
// small row is summed in fp64 and rounded once, in the order of the entries of A but for what the lanes of a long sum have, which
// is added up by halves.  A heavy entry is summed in integers where every partial sum is
// exact in them (all products are multiples of a power of two that the operands' values say; then the order of the additions
// does not matter and a whole block shares the accumulator), and otherwise in fp64 by one wave, entry after entry of A or four
// at a time.
#include "common.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace tsp {

constexpr int kPlanBlocks = 256;         // blocks that add up tile-rows, at most
constexpr int64_t kFinishRows = 1 << 21; // rows of which k_row_finish makes row_ptr (every block reads all groups before it)
constexpr int kChunkTileRows = 128, kChunkRows = kChunkTileRows * T;   // rows whose row_ptr one block writes
// Rows whose entries k_row_small adds up, and where: additions to one line wait for each other
constexpr int kPartTileRows = 128, kPartRows = kPartTileRows * T, kPartStride = 32;
constexpr int kPlanSums = 8;
constexpr int kSpanWindowsLog = 6, kSpanWindows = 1 << kSpanWindowsLog;   // windows whose bits the LDS of a block of k_heavy_count holds (32 KB)
constexpr int kGroupWindows = 4;         // tasks begin at a multiple of this many windows, those of very long rows of A at any
constexpr int kCountThreads = 256, kCountThreadsWide = 512;   // of k_heavy_count, and where four of its blocks fill the LDS
constexpr int kLongRow = 512;            // entries, for the threads that k_row_prepare gives a tile-row
constexpr int64_t kFoundEntries = (int64_t)2 << 30;   // of the small rows before they are moved into C, at most
// Intermediate products behind one task of k_heavy_fill (a row, or some of its windows), and entries of the row of A times
// windows: every step of a task goes through all entries, however few of them have anything in its windows.  (A row of 45,000
// entries among 100,000 of two, values in (-1, 1): 29 ms in one task of 25 windows, 3.4 in one each; by tiles 5.3.)
constexpr int kTaskProducts = 65536;
constexpr int kTaskEntries = 32768;

// Of a tile-row: the entries of its longest heavy row (23 bits hold the columns that k_row_prepare allows), its small rows,
// and the rows of 9 to 16 entries with no more products than a small row has; of either at most 16.
__host__ __device__ constexpr uint32_t pack_rows(uint32_t longest, uint32_t small, uint32_t wide) { return longest << 9 | (small * 17u + wide); }

struct RowMatrix {                       // an operand in the form the row kernels read
    // int32[rows + 1], clamped to [0, nnz] and non-decreasing inside a tile-row (16 rows and the start of the next), whatever
    // the operand holds: rows take no other entries than k_row_prepare has counted for them
    int32_t *start = nullptr;
    int2 *rec = nullptr;                 // per entry {column (clamped), value rounded to fp16, as fp32 bits}
    int32_t *ntiles = nullptr;           // tiles of every tile-row
    int32_t *tile_col = nullptr;         // their columns, at the position of the tile-row's first entry; any order
    uint32_t *range = nullptr;           // magnitude and granularity of every tile-row's values (ValueRange)
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
    // of A only (ub null for B):
    int32_t *ub;                         // products per row
    unsigned long long *products;        // ... per tile-row
    const void *b_row_ptr;               // of B, as the caller gave it
    int b_is_i64;
    int64_t b_rows;
    int32_t b_nnz;
    int small_lanes, small_products;     // most entries and products of a small row of A
    int windows;                         // of columns of C, for the heavy rows
    int32_t *heavy;                      // rows that are not small
    // {row, index into heavy, first window, one past the last window}; of rows of large_products and more from the front on,
    // of the others from the back.  (The tile-rows of the longest rows are done last, so that the kernels take the large tasks
    // from the last one on: R-MAT scale 14 sizing and multiplication of the large rows 49 + 94 -> 35 + 66 us, scale 18
    // 3.8 + 10.3 -> 3.4 + 9.8 ms.)
    int4 *tasks;
    int large_products;
    int64_t heavy_cap, task_cap;
    uint32_t *rows_of;                   // of every tile-row: pack_rows()
    uint32_t *part_len;                  // SmallArgs', zeroed; or null
    int64_t *d_scalars;
    const int64_t *skip;                 // S_ROW_SKIP, or null
};

__device__ __forceinline__ uint32_t half_bits(uint16_t bits) { return bits; }
__device__ __forceinline__ uint32_t half_bits(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }

// What a set of fp16 values spans: {256 + e} << 16 | {256 - g}, every |v| < 2^e and a multiple of 2^g; infinities and NaNs
// are as large as can be, zeros are left out.  The larger of each half over two sets holds for both.  ValueRange goes
// through the values of a set: the largest |v|, and the least exponent of a last bit (plus 25).
struct ValueRange {
    uint32_t most = 0, last = 1u << 20;
    __device__ __forceinline__ void take(uint32_t bits) {
        const uint32_t x = bits & 0x7FFFu, e = max(x >> 10, 1u);
        const uint32_t m = (x & 0x3FFu) | (x >= 0x400u ? 0x400u : 0u) | ((x - 1u) & 0x80000000u);
        most = max(most, x);
        last = min(last, e + (uint32_t)__builtin_ctz(m));
    }
    static __device__ __forceinline__ uint32_t range(uint32_t most, uint32_t last) {
        if (most == 0) return 0;
        if (most >= 0x7C00u) return 0x03FF03FFu;
        const int exponent = (int)(__float_as_uint((float)__builtin_bit_cast(_Float16, (uint16_t)most)) >> 23);
        return (uint32_t)(256 + exponent - 126) << 16 | (256u + 25u - last);
    }
};
__device__ __forceinline__ uint32_t range_max(uint32_t x, uint32_t y) {
    return max(x & 0xFFFF0000u, y & 0xFFFF0000u) | max(x & 0xFFFFu, y & 0xFFFFu);
}

__device__ __forceinline__ bool small_row(int32_t entries, int32_t products, int most_entries, int most_products) {
    return entries <= most_entries && products <= most_products;
}

// A team of kTeam threads per tile-row (a wave, or a block for long tile-rows), its entries flat over the lanes, kU of
// them per lane in flight.  The team's bitmap over the tile columns tells the first entry that falls into a tile (the
// atomic returns the word before): those lanes list the tile.  At the end a lane per row of A says whether the row is
// small or heavy and lists the heavy one with its tasks.
// Both operands at once (Second not empty) where they are of the same types and take teams of the same size: neither pass
// needs the other, and one behind the other each waits for its own way to memory and for its last blocks.  A*P on a 64^3 grid
// 19 + 10 -> 25 us, 4099 rows of 37 entries times as many 11 + 6 -> 11.
constexpr int prepare_teams(int team) { return team > 256 ? 1 : 256 / team; }     // in a block
struct NoSecond {};
template <typename RP, typename VT>
struct Second {
    PrepareArgs<RP, VT> args;
    uint32_t from;                       // the blocks from this one on are for it
};
template <int kTeam, int kU, typename RP, typename VT, typename Other = NoSecond>
__global__ __launch_bounds__(kTeam > 256 ? kTeam : 256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_row_prepare(const PrepareArgs<RP, VT> operand, const Other other) {
    constexpr int kTeams = prepare_teams(kTeam);
    constexpr bool kBoth = !std::is_same<Other, NoSecond>::value;
    typename std::conditional<kBoth, PrepareArgs<RP, VT>, const PrepareArgs<RP, VT> &>::type a = operand;
    uint32_t block = blockIdx.x;
    if constexpr (kBoth)
        if (block >= other.from) {
            a = other.args;
            block -= other.from;
        }
    if (a.skip && uniform_load(a.skip)) return;
    extern __shared__ uint32_t lds_bitmap[];
    __shared__ int32_t s_ptr[kTeams][T + 1];
    __shared__ unsigned long long s_ub[kTeams][T];
    __shared__ int32_t s_count[kTeams];
    __shared__ uint32_t s_most[kTeams], s_last[kTeams];
    const int team = threadIdx.x / kTeam, tid = threadIdx.x % kTeam, lane = lane_id();
    uint32_t *bitmap = lds_bitmap + team * a.bitmap_words;
    const int64_t tile_rows = (a.rows + T - 1) / T;
    const int64_t I = (int64_t)block * kTeams + team;
    const bool live = I < tile_rows;
    bool bad = false;
    if (live) {
        for (int w = tid; w < a.bitmap_words / 4; w += kTeam) reinterpret_cast<uint4 *>(bitmap)[w] = make_uint4(0, 0, 0, 0);
        if (tid <= T) {
            const int64_t i = min(I * T + tid, a.rows);
            const RP raw = a.row_ptr[i];
            int32_t p = (int32_t)min(max(raw, (RP)0), (RP)a.nnz);
            p = max(p, TSP_DPP(p, p, 0x111, 0xf, false));
            p = max(p, TSP_DPP(p, p, 0x112, 0xf, false));
            p = max(p, TSP_DPP(p, p, 0x114, 0xf, false));
            p = max(p, TSP_DPP(p, p, 0x118, 0xf, false));
            p = max(p, TSP_DPP(p, p, 0x142, 0xa, false));
            bad = raw != (RP)p || (i == 0 && raw != 0) || (i == a.rows && raw != (RP)a.nnz);
            s_ptr[team][tid] = p;
            if (tid < T) s_ub[team][tid] = 0;
            if (i < a.rows ? tid < T : true) a.out.start[i] = p;
        }
        if (tid == 0) {
            s_count[team] = 0;
            s_most[team] = 0;
            s_last[team] = 1u << 20;
        }
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (live) {
        const int32_t e0 = s_ptr[team][0], e1 = s_ptr[team][T];
        int32_t listed = 0;
        ValueRange range;
        int32_t c[kU], prev[kU];
        VT v[kU];
        auto request = [&](int32_t base) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int32_t k = min(base + u * kTeam + lane, e1 - 1);
                c[u] = a.col[k];
                prev[u] = a.col[max(k - 1, 0)];
                v[u] = a.val[k];
            }
        };
        int32_t base = e0 + (tid & ~63);
        if (base < e1) request(base);
        for (; base < e1; base += kTeam * kU) {
            // (every part for all entries in flight before the next part: look-ups and additions to LDS one behind the other
            // made a trip of a long tile-row twice as long)
            int32_t len[kU];
            int r[kU];
            bool first[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                bad = bad || (uint32_t)c[u] >= (uint64_t)a.cols;
                if ((uint32_t)c[u] >= (uint64_t)a.cols) c[u] = 0;
                len[u] = 0;
                if (a.ub && c[u] < a.b_rows) {
                    // (no less than B's own start array will say, which is clamped the same and then made non-decreasing)
                    int32_t s, e;
                    if (a.b_is_i64) {
                        s = (int32_t)min(max(static_cast<const int64_t *>(a.b_row_ptr)[c[u]], (int64_t)0), (int64_t)a.b_nnz);
                        e = (int32_t)min(max(static_cast<const int64_t *>(a.b_row_ptr)[c[u] + 1], (int64_t)0), (int64_t)a.b_nnz);
                    } else {
                        s = min(max(static_cast<const int32_t *>(a.b_row_ptr)[c[u]], 0), a.b_nnz);
                        e = min(max(static_cast<const int32_t *>(a.b_row_ptr)[c[u] + 1], 0), a.b_nnz);
                    }
                    len[u] = min(max(e - s, 0), (1 << 25) - 1);
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) r[u] = 0;
#pragma unroll
            for (int step = T / 2; step >= 1; step >>= 1)
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if (s_ptr[team][r[u] + step] <= base + u * kTeam + lane) r[u] += step;
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int32_t k = base + u * kTeam + lane;
                const bool on = k < e1, starts = k == s_ptr[team][r[u]];
                bad = bad || (on && !starts && prev[u] >= c[u]);
                if (on) {
                    const uint32_t bits = half_bits(v[u]);
                    a.out.rec[k] = make_int2(c[u], (int)__float_as_uint((float)__builtin_bit_cast(_Float16, (uint16_t)bits)));
                    range.take(bits);
                }
                first[u] = on && (starts || (prev[u] >> 4) != (c[u] >> 4));
            }
            uint32_t had[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int32_t t = c[u] >> 4;
                had[u] = first[u] ? atomicOr(&bitmap[t >> 5], 1u << (t & 31)) : 0u;
            }
            int32_t tile[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                tile[u] = c[u] >> 4;
                first[u] = first[u] && !((had[u] >> (tile[u] & 31)) & 1u);
            }
            const int32_t next = base + kTeam * kU;
            if (next < e1) request(next);
            int32_t at = listed, found = 0;
            unsigned long long firsts[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                firsts[u] = __ballot(first[u]);
                found += __popcll(firsts[u]);
            }
            if constexpr (kTeam == 64) {
                listed += found;
            } else if (found) {
                if (lane == 0) at = atomicAdd(&s_count[team], found);
                at = __builtin_amdgcn_readfirstlane(at);
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (first[u]) a.out.tile_col[e0 + at + __popcll(firsts[u] & ((1ull << lane) - 1ull))] = tile[u];
                at += __popcll(firsts[u]);
            }
            if (a.ub && kTeam == 64) {
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if (base + u * kTeam + lane < e1) atomicAdd(&s_ub[team][r[u]], (unsigned long long)(uint32_t)len[u]);    // (rows of few entries)
            } else if (a.ub) {
                // products per row: differences of the running sum at the ends of the rows' stretches in this wave
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    if (base + u * kTeam >= e1) break;               // (the whole wave)
                    const bool on = base + u * kTeam + lane < e1;
                    const uint32_t mine = on ? (uint32_t)len[u] : 0u, inc = wave_inclusive_scan(mine);
                    const int r_next = __shfl_down(r[u], 1, 64), r_prev = __shfl_up(r[u], 1, 64);
                    if (on && (lane == 63 || r_next != r[u] || base + u * kTeam + lane == e1 - 1)) atomicAdd(&s_ub[team][r[u]], (unsigned long long)inc);
                    if (on && lane > 0 && r_prev != r[u])
                        atomicAdd(&s_ub[team][r[u]], (unsigned long long)0 - (unsigned long long)(inc - mine));
                }
            }
        }
        const int most = wave_max((int)range.most), last = -wave_max(-(int)range.last);
        if (lane == 0) {
            if constexpr (kTeam == 64) s_count[team] = listed;
            atomicMax(&s_most[team], (uint32_t)most);
            atomicMin(&s_last[team], (uint32_t)last);
        }
    }
    if constexpr (kTeam == 64) wave_sync();
    else __syncthreads();
    if (!live) return;
    if (bad && a.validate) a.d_scalars[S_INVALID] = 1;
    if (tid == 0) {
        a.out.ntiles[I] = s_count[team];
        if (a.ub && a.part_len && I % kPartTileRows == 0) a.part_len[I / kPartTileRows * kPartStride] = 0;
        a.out.range[I] = ValueRange::range(s_most[team], s_last[team]);
    }
    if (!a.ub || tid >= 64) return;
    // a lane per row
    const int64_t row = I * T + tid;
    int tasks = 0, deg = 0;
    unsigned long long ub = 0;
    const int groups = (a.windows + kGroupWindows - 1) / kGroupWindows;
    if (tid < T && row < a.rows) {
        ub = min(s_ub[team][tid], (unsigned long long)INT32_MAX);
        deg = s_ptr[team][tid + 1] - s_ptr[team][tid];
        a.ub[row] = (int32_t)ub;
        if (deg > 0 && ub > 0 && !small_row(deg, (int32_t)ub, a.small_lanes, a.small_products))
            tasks = max(min(max((int)ub / kTaskProducts, 1), groups), (int)min((int64_t)deg * a.windows / kTaskEntries, (int64_t)a.windows));
    }
    unsigned long long all = tid < T ? s_ub[team][tid] : 0ull;
    for (int d = 1; d < T; d <<= 1) all += __shfl_xor(all, d, T);
    if (tid == 0) a.products[I] = all;
    const unsigned long long heavies = __ballot(tasks > 0);
    if (heavies) {                       // places in both lists from one atomic, and from another for the large ones
        const bool large = ub >= (unsigned long long)a.large_products;
        const uint32_t light_inc = wave_inclusive_scan(large ? 0u : (uint32_t)tasks), large_inc = wave_inclusive_scan(large ? (uint32_t)tasks : 0u);
        unsigned long long at = 0, large_at = 0;
        if (lane == 63) {
            at = atomicAdd(reinterpret_cast<unsigned long long *>(a.d_scalars + S_ROW_LISTS),
                           ((unsigned long long)__popcll(heavies) << 36) | light_inc);
            if (large_inc) large_at = atomicAdd(reinterpret_cast<unsigned long long *>(a.d_scalars + S_ROW_LARGE_TASKS), (unsigned long long)large_inc);
        }
        at = __shfl(at, 63, 64);
        large_at = __shfl(large_at, 63, 64);
        const int64_t h = (int64_t)(at >> 36) + __popcll(heavies & ((1ull << lane) - 1ull));
        const int64_t t0 = large ? (int64_t)large_at + large_inc - tasks
                                : a.task_cap - ((int64_t)(at & ((1ull << 36) - 1ull)) + light_inc);
        if (tasks > 0 && h < a.heavy_cap) {
            a.heavy[h] = (int32_t)row;
            // (groups of windows, as even as they go; single ones where there are more tasks than groups)
            const int unit = tasks > groups ? 1 : kGroupWindows, units = tasks > groups ? a.windows : groups;
            for (int t = 0; t < tasks; ++t)
                if ((uint64_t)(t0 + t) < (uint64_t)a.task_cap)
                    a.tasks[t0 + t] = make_int4((int)row, (int)h, (int)((int64_t)units * t / tasks) * unit,
                                                min((int)((int64_t)units * (t + 1) / tasks) * unit, a.windows));
        }
    }
    const int longest = heavies ? wave_max(tasks > 0 ? deg : 0) : 0, small = __popcll(__ballot(deg > 0 && ub > 0 && tasks == 0));
    const int wide = __popcll(__ballot(deg > 8 && ub > 0 && small_row(deg, (int32_t)ub, 16, a.small_products)));
    if (lane == 0) a.rows_of[I] = pack_rows((uint32_t)min(longest, (1 << 23) - 1), (uint32_t)small, (uint32_t)wide);
}

// A store that a block of the same launch on another XCD can read (get_shared), past the L2 caches, which do not see each
// other's; plain otherwise.
template <typename X>
__device__ __forceinline__ void put_for(bool shared, X *p, X v) {
    if (shared) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
template <bool kShared, typename X>
__device__ __forceinline__ X get_shared(const X *p) {
    if constexpr (kShared) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}

// What the operands are like, summed over their tile-rows.  The blocks leave their sums in `partial`; k_row_finish, which
// runs after them, adds those up, or for products of a few rows the block of k_row_small that finishes last.  (With many
// blocks that takes too long: an addition per block to one counter is 9 ns, and device-wide fences write back the L2 caches:
// 90 us instead of 8 on a 512^2 mesh.)
struct SumArgs {
    int64_t a_tile_rows, b_tile_rows;
    const int32_t *a_start, *a_ntiles, *a_tile_col, *b_ntiles;
    const uint32_t *rows_of;
    const uint32_t *a_range, *b_range;
    const unsigned long long *products;
    int same;                            // A and B are one matrix
    unsigned long long *partial;         // [kPlanSums][kPlanBlocks]
    const int64_t *skip;                 // S_ROW_SKIP, or null
};
enum { kSumCandidates, kSumTilesA, kSumTilesB, kSumProducts, kSumSmall, kSumRanges, kSumLongest, kSumWide };

// Sixteen lanes per tile-row: tiles, candidate pairs (the tiles of B's tile-rows behind the tiles of A: the measure by
// which tsp_spgemm chooses this path), products, value ranges.
// `shared`: another block of this launch reads the sums.
__device__ __forceinline__ void sum_tile_rows(const SumArgs &a, int block, int blocks, bool shared = false) {
    __shared__ unsigned long long s_sum[kPlanSums], s_max[kPlanSums];
    const int lane = lane_id(), r = threadIdx.x & 15;
    if (threadIdx.x < kPlanSums) s_sum[threadIdx.x] = s_max[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long cand = 0, tiles_a = 0, tiles_b = 0, products = 0, small = 0, wide = 0;
    uint32_t range_a = 0, range_b = 0;
    int longest = 0;
    const int64_t most = max(a.a_tile_rows, a.same ? (int64_t)0 : a.b_tile_rows);
    // (neighbours to different blocks, and of a block's tile-rows one to each wave first: the tile-rows of the hubs of a graph
    // lie side by side, and one by one they kept the launch waiting for 290 us on R-MAT scale 18)
    const int at = (threadIdx.x >> 6) + 4 * ((threadIdx.x >> 4) & 3);
    for (int64_t base = block; base < most; base += (int64_t)blocks * 16) {
        const int64_t I = base + (int64_t)at * blocks;
        if (r == 0 && I < a.b_tile_rows && !a.same) {
            tiles_b += (unsigned)a.b_ntiles[I];
            range_b = range_max(range_b, a.b_range[I]);
        }
        int32_t e0 = 0, n = 0;
        if (I < a.a_tile_rows) {
            e0 = a.a_start[I * T];
            n = a.a_ntiles[I];
            if (r == 0) {
                tiles_a += (unsigned)n;
                range_a = range_max(range_a, a.a_range[I]);
                products += a.products[I];
                const uint32_t rows_of = a.rows_of[I], rows = rows_of & 511u;
                longest = max(longest, (int)(rows_of >> 9));
                small += rows / 17u;
                wide += rows % 17u;
            }
            for (int32_t j = r; j < min(n, 128); j += 64) {
                int32_t K[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) K[u] = a.a_tile_col[e0 + min(j + 16 * u, n - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j + 16 * u < n && K[u] < a.b_tile_rows) cand += (unsigned)a.b_ntiles[K[u]];
            }
        }
        // long tile-rows: the rest of their tiles by the whole wave
        for (unsigned long long more = __ballot(r == 0 && n > 128); more; more &= more - 1) {
            const int from = __ffsll((long long)more) - 1;
            const int32_t first = __builtin_amdgcn_readlane(e0, from), count = __builtin_amdgcn_readlane(n, from);
            for (int32_t j = 128 + lane; j < count; j += 256) {
                int32_t K[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) K[u] = a.a_tile_col[first + min(j + 64 * u, count - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j + 64 * u < count && K[u] < a.b_tile_rows) cand += (unsigned)a.b_ntiles[K[u]];
            }
        }
    }
    auto add = [&](int slot, unsigned long long v) {
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (lane == 0 && v) atomicAdd(&s_sum[slot], v);
    };
    add(kSumCandidates, cand);
    add(kSumTilesA, tiles_a);
    add(kSumTilesB, tiles_b);
    add(kSumProducts, products);
    add(kSumSmall, small);
    add(kSumWide, wide);
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
    if (threadIdx.x == 0) {
        s_sum[kSumRanges] = s_max[0] << 48 | s_max[1] << 32 | s_max[2] << 16 | s_max[3];
        s_sum[kSumLongest] = s_max[4];
    }
    __syncthreads();
    if (threadIdx.x < kPlanSums) put_for(shared, &a.partial[threadIdx.x * kPlanBlocks + block], s_sum[threadIdx.x]);
}
__global__ __launch_bounds__(256) void k_row_sums(const SumArgs a) {
    if (a.skip && uniform_load(a.skip)) return;
    sum_tile_rows(a, blockIdx.x, gridDim.x);
}

// The accumulator that is exact for the heavy rows: int32_t, long long or double; the integers are values times 2^-scale.
struct FillKind {
    enum Sum : int { kInt32, kInt64, kDouble } sum;
    int scale;
};
// Bits of the operands' values as integers (multiples of their common granularity), and of a sum of as many products as
// the longest heavy row of A has entries, if those are the integers of `scale`.
__host__ __device__ inline bool fill_exact(FillKind k, int64_t range_a, int64_t range_b, int64_t longest) {
    if (k.sum == FillKind::kDouble) return true;
    const int ra = (int)range_a, rb = (int)range_b;
    if (!ra || !rb || (ra >> 16) >= 1023 || (rb >> 16) >= 1023) return false;
    const int product_bits = (ra >> 16) + (rb >> 16) - 512 - k.scale, granularity = 512 - (ra & 0xFFFF) - (rb & 0xFFFF);
    int bits = product_bits;
    for (int64_t n = 1; n < longest; n <<= 1) ++bits;
    return granularity >= k.scale && (k.sum == FillKind::kInt32 ? bits <= 31 : bits <= 63 && product_bits <= 51);
}
__host__ __device__ inline FillKind fill_kind(const int64_t *h) {
    const int scale = 512 - (int)(h[S_ROW_RANGE_A] & 0xFFFF) - (int)(h[S_ROW_RANGE_B] & 0xFFFF);
    for (auto sum : {FillKind::kInt32, FillKind::kInt64})
        if (fill_exact({sum, scale}, h[S_ROW_RANGE_A], h[S_ROW_RANGE_B], h[S_ROW_LONGEST])) return {sum, scale};
    return {FillKind::kDouble, 0};
}

// What the kernels of the multiplication have been launched with before the host knows the sizes
struct Expected {
    int64_t nnz, heavy, tasks, large;
    FillKind kind;
    __host__ __device__ bool holds(const int64_t *scalars) const {
        return !scalars[S_INVALID] && scalars[S_C_NNZ] <= nnz && scalars[S_ROW_HEAVY] <= heavy && scalars[S_ROW_TASKS] - scalars[S_ROW_LARGE_TASKS] <= tasks - large &&
               scalars[S_ROW_LARGE_TASKS] <= large &&
               fill_exact(kind, scalars[S_ROW_RANGE_A], scalars[S_ROW_RANGE_B], scalars[S_ROW_LONGEST]) &&
               // (fp64 does for any values, but where integers do their sums have other last bits)
               (kind.sum != FillKind::kDouble || fill_kind(scalars).sum == FillKind::kDouble);
    }
};

struct FinishArgs {
    int64_t rows;                        // 0: only the sizes are wanted
    const int32_t *row_nnz;
    const uint32_t *group_len;           // sums of row_nnz over 16 rows, padded to a multiple of four
    int64_t *c_row_ptr;
    const unsigned long long *partial;   // of k_row_sums
    int partials, same;
    int64_t *d_scalars, *h_scalars_dev;
    int64_t publish_tag;
    bool clear;                          // the scalar block, for the next call
    Expected expected;
    int32_t *live;                       // [3]: whether what is expected holds, and the numbers of all and of the large tasks
    const int64_t *skip;                 // S_ROW_SKIP, or null: nothing has been counted then
};

// What one block that knows that the others are done makes of the sums over the tile-rows, and all sizes to the host.
// `standing`: standing_scalar; `entries`: of C, where rows > 0.
struct PlanTotals {
    unsigned long long sum[kPlanSums], most[kPlanSums];
    int64_t own[kScalars];
};
template <bool kShared>
__device__ __forceinline__ void add_plan_sums(const FinishArgs &a, PlanTotals &totals) {       // (two sums per wave)
    const int lane = lane_id(), slot0 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 2;
    unsigned long long v[2][kPlanBlocks / 64];                   // (both requested before either is waited for)
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int u = 0; u < kPlanBlocks / 64; ++u)
            v[w][u] = u * 64 + lane < a.partials ? get_shared<kShared>(a.partial + (slot0 + w) * kPlanBlocks + u * 64 + lane) : 0ull;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int slot = slot0 + w;
        if (slot == kSumRanges || slot == kSumLongest) {
            int most[4] = {0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < kPlanBlocks / 64; ++u) {
                if (slot == kSumLongest) most[0] = max(most[0], (int)v[w][u]);
                else
                    for (int q = 0; q < 4; ++q) most[q] = max(most[q], (int)((v[w][u] >> (48 - 16 * q)) & 0xFFFFull));
            }
            for (int q = 0; q < 4; ++q) most[q] = wave_max(most[q]);
            if (lane == 0)
                for (int q = 0; q < (slot == kSumLongest ? 1 : 4); ++q) totals.most[slot == kSumLongest ? 4 : q] = (unsigned long long)most[q];
        } else {
            unsigned long long sum = 0;
#pragma unroll
            for (int u = 0; u < kPlanBlocks / 64; ++u) sum += v[w][u];
            for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
            if (lane == 0) totals.sum[slot] = sum;
        }
    }
    __syncthreads();
}
__device__ __forceinline__ void publish_sizes(const FinishArgs &a, PlanTotals &totals, int64_t standing, int64_t entries) {
    int64_t *own = totals.own;
    const unsigned long long *s_sum = totals.sum, *s_max = totals.most;
    if (threadIdx.x == S_C_NNZ) own[S_C_NNZ] = a.rows > 0 ? entries : standing;
    if (threadIdx.x == S_INVALID) own[S_INVALID] = standing;
    if (threadIdx.x == S_ROW_LISTS || threadIdx.x == S_ROW_LARGE_TASKS) own[threadIdx.x] = standing;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (a.rows > 0) a.c_row_ptr[a.rows] = entries;
        own[S_CANDIDATES] = (int64_t)s_sum[kSumCandidates];
        own[S_TILES_A] = (int64_t)s_sum[kSumTilesA];
        own[S_TILES_B] = (int64_t)(a.same ? s_sum[kSumTilesA] : s_sum[kSumTilesB]);
        own[S_ROW_PRODUCTS] = (int64_t)s_sum[kSumProducts];
        own[S_ROW_SMALL] = (int64_t)s_sum[kSumSmall];
        own[S_ROW_WIDE] = (int64_t)s_sum[kSumWide];
        const int from = a.same ? 0 : 2;
        own[S_ROW_RANGE_A] = (int64_t)(s_max[0] << 16 | s_max[1]);
        own[S_ROW_RANGE_B] = (int64_t)(s_max[from] << 16 | s_max[from + 1]);
        own[S_ROW_LONGEST] = (int64_t)s_max[4];
        const unsigned long long lists = (unsigned long long)own[S_ROW_LISTS];
        own[S_ROW_HEAVY] = (int64_t)(lists >> 36);
        own[S_ROW_TASKS] = (int64_t)(lists & ((1ull << 36) - 1ull)) + own[S_ROW_LARGE_TASKS];
        if (a.live) {
            a.live[0] = a.expected.holds(own);
            a.live[1] = (int32_t)own[S_ROW_TASKS];
            a.live[2] = (int32_t)own[S_ROW_LARGE_TASKS];
        }
    }
    constexpr uint32_t kOwn = own_slot(S_C_NNZ) | own_slot(S_CANDIDATES) | own_slot(S_TILES_A) | own_slot(S_TILES_B) |
                              own_slot(S_ROW_PRODUCTS) | own_slot(S_ROW_SMALL) | own_slot(S_ROW_WIDE) | own_slot(S_ROW_RANGE_A) | own_slot(S_ROW_RANGE_B) |
                              own_slot(S_ROW_LONGEST) | own_slot(S_ROW_HEAVY) | own_slot(S_ROW_TASKS);
    publish_scalars(a.d_scalars, a.h_scalars_dev, a.publish_tag, standing, own, kOwn, a.clear);
}

// row_ptr of C from the row lengths: block b takes rows [2048 b, 2048 b + 2048), adds up the groups of 16 rows before
// them and scans its own.  The last block also adds up the sums over the tile-rows and hands all sizes to the host.
// kShared: other blocks of the same launch have left row_nnz and partial (put_for).
template <bool kShared>
__device__ __forceinline__ void row_finish(const FinishArgs &a, int block, int blocks) {
    __shared__ uint64_t lds[256 / 64];
    __shared__ PlanTotals totals;
    const bool last = block == blocks - 1;
    const int64_t standing = last ? standing_scalar(a.d_scalars) : 0;
    constexpr int kItems = kChunkRows / 256;
    const int64_t base = (int64_t)block * kChunkRows + (int64_t)threadIdx.x * kItems;
    int32_t x[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) x[i] = base + i < a.rows ? get_shared<kShared>(a.row_nnz + base + i) : 0;
    if (last) add_plan_sums<kShared>(a, totals);
    uint64_t before = 0;
    const uint4 *groups4 = reinterpret_cast<const uint4 *>(a.group_len);
    const int64_t quads = a.rows > 0 ? (int64_t)block * kChunkTileRows / 4 : 0;
    // (all of them in flight up to 16384 groups: a round trip, not four)
    for (int64_t q0 = threadIdx.x; q0 < quads; q0 += 16 * 256) {
        uint4 g[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) g[u] = groups4[min(q0 + u * 256, quads - 1)];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (q0 + u * 256 < quads) before += (uint64_t)g[u].x + g[u].y + g[u].z + g[u].w;
    }
    uint64_t entries_before = 0;
    if (block > 0) (void)block_exclusive_scan64<256>(before, &entries_before, lds);
    uint64_t mine = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) mine += (uint32_t)x[i];
    uint64_t total;
    uint64_t run = entries_before + block_exclusive_scan64<256>(mine, &total, lds);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (base + i < a.rows) a.c_row_ptr[base + i] = (int64_t)run;
        run += (uint32_t)x[i];
    }
    if (last) publish_sizes(a, totals, standing, (int64_t)(entries_before + total));
}
__global__ __launch_bounds__(256) void k_row_finish(const FinishArgs a) {
    if (a.skip && uniform_load(a.skip)) publish_scalars(a.d_scalars, a.h_scalars_dev, a.publish_tag, standing_scalar(a.d_scalars), nullptr, 0);
    else row_finish<false>(a, blockIdx.x, gridDim.x);
}

// ---- small rows -------------------------------------------------------------------------------------------------
// How the small rows of a launch are worked off: lanes per row of A, lanes per row of B (a power of two, at most as
// many), and the most products of a small row: 24, 48, 96 or 192, three quarters of the keys that the group sorts then.  (From a hash
// table that was to stay that empty; the sort would take the last quarter at the same price, which has not been timed.)
struct SmallShape {
    int lanes, list_lanes, products;
    bool narrow() const { return list_lanes < lanes; }
    int wave_rows() const { return 64 / lanes; }
    size_t wave_bytes() const { return (size_t)(wave_rows() * products + 2) * 8; }   // LDS
    static constexpr size_t kReadPast = 64 * 8;              // ... behind the last wave's
};

struct SmallArgs {
    SmallShape shape;
    int wave_bytes;
    int64_t rows;
    int32_t *row_nnz;
    uint32_t *group_len;                 // entries per 16 rows
    // For k_small_finish, or null: entries per part of kPartRows, zero before, and whether the operands are canonical and no
    // row is heavy
    uint32_t *part_len;
    int32_t *only_small;
    const int64_t *d_scalars;
    uint32_t *block_len;                 // GivenOperands: entries of a block's rows
    int2 *found;                         // [waves][wave_rows * products] entries {column, value} of a wave's rows, in order
    int32_t *wave_total;                 // ... and how many
    // The blocks that sum (SumArgs) are the first ones of the launch where their groups of lanes have several tile-rows each, else
    // the last ones, which fill what the rows leave of the chip: R-MAT scale 18 490 us behind the rows, 300 before them, A*P on a
    // 64^3 grid 29 and 24; 65,536 rows of 8 random entries 44 and 47.
    int sum_blocks;
    bool sums_first;
    int finish;                          // the last block does the work of k_row_finish (FinishArgs; rows of one chunk)
};

// Where k_row_small finds its rows: as k_row_prepare has left the operands.  list: entry l of a row of A, if it is small and has one:
// its value as fp32 bits, and where its row of B lies; of GivenOperands also whether the row has more than 8 entries.  element: an
// entry of B, as it is read and as {column, value as fp32 bits}.
struct PreparedOperands {
    const int32_t *a_start, *b_start, *ub;
    const int2 *a_rec, *b_rec;
    static constexpr bool kDirect = false;
    using Element = int2;
    template <int G>
    __device__ __forceinline__ void list(uint32_t row, int l, int most, int32_t &p, int32_t &e, uint32_t &value, bool &other, bool &) const {
        const int32_t s = element(a_start, row), deg = element(a_start, row + 1) - s, products = element(ub, row);
        const bool small = (products > 0) & (deg > 0) & small_row(deg, products, G, most);
        other = !small & (products != 0) & (deg > 0);
        if (small & (l < deg)) {
            const int2 x = element(a_rec, (uint32_t)(s + l));
            p = element(b_start, (uint32_t)x.x);
            e = element(b_start, (uint32_t)x.x + 1);
            value = (uint32_t)x.y;
        }
    }
    __device__ __forceinline__ Element read(uint32_t k) const {
        uint32_t byte = k * 8u;
        asm volatile("" : "+v"(byte));                       // (a 32-bit offset from a scalar base)
        return *reinterpret_cast<const int2 *>(reinterpret_cast<const char *>(b_rec) + byte);
    }
    __device__ __forceinline__ int2 entry(const Element &x) const { return x; }
};
// ... or as the caller gave them, of the same types; nothing is read outside their arrays whatever they hold.  Reading columns and
// values apart takes k_row_small of a 512 x 512 mesh 29.5 us instead of 28.3, and spares the pass that puts them together (16).
template <typename RP, typename VT>
struct GivenOperands {
    const RP *a_row_ptr, *b_row_ptr;
    const int32_t *a_col, *b_col;
    const VT *a_val, *b_val;
    int32_t a_nnz, b_nnz;
    uint32_t a_last, b_last;                                 // columns, less one
    static constexpr bool kDirect = true;
    struct Element {
        int32_t col;
        VT val;
    };
    static __device__ __forceinline__ int32_t pointer(const RP *row_ptr, uint32_t row, int32_t nnz) {
        return (int32_t)min(max(element(row_ptr, row), (RP)0), (RP)nnz);
    }
    static __device__ __forceinline__ uint32_t value_bits(VT v) { return __float_as_uint((float)__builtin_bit_cast(_Float16, (uint16_t)half_bits(v))); }
    template <int G>
    __device__ __forceinline__ void list(uint32_t row, int l, int, int32_t &p, int32_t &e, uint32_t &value, bool &other, bool &wide) const {
        const int32_t s = pointer(a_row_ptr, row, a_nnz), deg = pointer(a_row_ptr, row + 1, a_nnz) - s;
        other = deg > G;
        wide = deg > 8;
        if (!other & (l < deg)) {
            const uint32_t c = min((uint32_t)element(a_col, (uint32_t)(s + l)), a_last);
            value = value_bits(element(a_val, (uint32_t)(s + l)));
            p = pointer(b_row_ptr, c, b_nnz);
            e = pointer(b_row_ptr, c + 1, b_nnz);
        }
    }
    __device__ __forceinline__ Element read(uint32_t k) const {
        uint32_t byte = k * (uint32_t)sizeof(VT);
        asm volatile("" : "+v"(byte));
        return {*reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(b_col) + byte * (4u / (uint32_t)sizeof(VT))),
                *reinterpret_cast<const VT *>(reinterpret_cast<const char *>(b_val) + byte)};
    }
    __device__ __forceinline__ int2 entry(const Element &x) const { return make_int2((int)min((uint32_t)x.col, b_last), (int)value_bits(x.val)); }
};

// The wave's groups of G lanes each sort G * R keys, number l * R + r of a group in lane l's key[r]: merges of ascending halves,
// of which the first step compares mirrored places, so that every step puts the smaller key first and no lane needs to know a
// direction.  med3 with 0 is a minimum, with the largest number a maximum.  (Templates, not loops: sixteen keys are too many for the
// compiler to take the loops apart, and then all lie in scratch memory.  As it is, the 64 registers that leave room for eight waves
// are too few for sixteen keys by 9 to 12, which are stored and read back around that sort; rows of up to 128 products have none of
// it but for one register of k_row_given with lists of tiles.)
template <int kControl>
__device__ __forceinline__ uint32_t from_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kControl, 0xf, 0xf, true); }
template <int kXor>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t x) {
    if constexpr (kXor == 1) return from_lane<0xB1>(x);
    else if constexpr (kXor == 2) return from_lane<0x4E>(x);
    else if constexpr (kXor == 3) return from_lane<0x1B>(x);
    else if constexpr (kXor == 4) return from_lane<0x1B>(from_lane<0x141>(x));
    else if constexpr (kXor == 7) return from_lane<0x141>(x);
    else if constexpr (kXor == 15) return from_lane<0x140>(x);
    else static_assert(kXor == 1, "not needed");
}
__device__ __forceinline__ uint32_t median(uint32_t x, uint32_t y, uint32_t z) {
    return max(min(x, y), min(max(x, y), z));                // (v_med3_u32)
}
template <int R, int kStride>
__device__ __forceinline__ void sort_strides(uint32_t (&key)[R]) {       // kStride, kStride / 2, ... 1
    if constexpr (kStride >= 1) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (!(r & kStride)) {
                const uint32_t x = min(key[r], key[r + kStride]);
                key[r + kStride] = max(key[r], key[r + kStride]);
                key[r] = x;
            }
        sort_strides<R, kStride / 2>(key);
    }
}
template <int R, int kSorted>
__device__ __forceinline__ void sort_own(uint32_t (&key)[R]) {           // stretches of kSorted keys are sorted
    if constexpr (kSorted < R) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (!(r & kSorted)) {
                const int other = r ^ (2 * kSorted - 1);
                const uint32_t x = min(key[r], key[other]);
                key[other] = max(key[r], key[other]);
                key[r] = x;
            }
        sort_strides<R, kSorted / 2>(key);
        sort_own<R, 2 * kSorted>(key);
    }
}
template <int kXor, bool kMirror, int R>
__device__ __forceinline__ void sort_across(uint32_t (&key)[R], uint32_t upper) {
    uint32_t other[R];
#pragma unroll
    for (int r = 0; r < R; ++r) other[r] = from_lane_xor<kXor>(key[kMirror ? r ^ (R - 1) : r]);
#pragma unroll
    for (int r = 0; r < R; ++r) key[r] = median(key[r], other[r], upper);
}
template <int G, int R>
__device__ __forceinline__ void sort_group(uint32_t (&key)[R], int l) {
    const uint32_t upper1 = l & 1 ? ~0u : 0u, upper2 = l & 2 ? ~0u : 0u, upper4 = l & 4 ? ~0u : 0u, upper8 = l & 8 ? ~0u : 0u;
    sort_own<R, 1>(key);
    sort_across<1, true>(key, upper1);
    sort_strides<R, R / 2>(key);
    sort_across<3, true>(key, upper2);
    sort_across<1, false>(key, upper1);
    sort_strides<R, R / 2>(key);
    sort_across<7, true>(key, upper4);
    sort_across<2, false>(key, upper2);
    sort_across<1, false>(key, upper1);
    sort_strides<R, R / 2>(key);
    if constexpr (G == 16) {
        sort_across<15, true>(key, upper8);
        sort_across<4, false>(key, upper4);
        sort_across<2, false>(key, upper2);
        sort_across<1, false>(key, upper1);
        sort_strides<R, R / 2>(key);
    }
}

// What the lane of each round's list holds: from one lane of the group to all of it, in the registers, or where a round has several
// lists through LDS.
template <bool kNarrow, int G, int kRound, typename OfList>
__device__ __forceinline__ int of_round(int v, OfList &of_list) {
    if constexpr (kNarrow) return of_list(v, kRound);
    else if constexpr (G == 16) return __builtin_amdgcn_mov_dpp(v, 0x150 + kRound, 0xf, 0xf, true);
    else return __builtin_amdgcn_update_dpp(__builtin_amdgcn_mov_dpp(v, 0x150 + kRound, 0xf, 0xf, true), v, 0x158 + kRound, 0xf, 0xc, false);
}
template <bool kNarrow, int G, int kFrom, typename OfList, int... kRound>
__device__ __forceinline__ void each_list(int *out, int v, OfList &of_list, std::integer_sequence<int, kRound...>) {
    ((out[kRound] = of_round<kNarrow, G, kFrom + kRound>(v, of_list)), ...);
}
template <int kFrom, int kTo, typename Run>
__device__ __forceinline__ void each_round(Run &run) {
    if constexpr (kFrom < kTo) {
        run(std::integral_constant<int, kFrom>{});
        each_round<kFrom + 1, kTo>(run);
    }
}
// The bits of the wave's groups of G lanes, one over the other
template <int G>
__device__ __forceinline__ uint32_t fold_groups(unsigned long long bits) {
    uint32_t x = (uint32_t)bits | (uint32_t)(bits >> 32);
    x |= x >> 16;
    if constexpr (G == 8) x |= x >> 8;
    return x & ((1u << G) - 1u);
}

// A group of G lanes per row of A with at most G entries and shape.products intermediate products.  The rows of B behind
// it are fetched by the group's lanes side by side (a lane per list costs the load path a cycle per lane), all before the
// first is used.  The products go to LDS, in the order of A's entries and behind them of B's; their keys {column << 8 | place} are
// sorted in the lanes' registers, and the products of a column, which then follow one another, are added up in fp64, in a lane one
// after the other and over the lanes by a scan.  The wave's rows go in order into memory of their own: k_small_copy moves them into
// C when its row_ptr is known.  (Doing all of it twice, once for the sizes, costs more than the copy.)
// A whole group per row of B (kNarrow false): one row of B at a time.  Short rows of B (kNarrow): several at a time.
// Bound by the round trips of a wave (row of A, its entries, the starts of B's rows, their entries) and the few waves that are there
// to hide them while a launch begins and ends; vector instructions 63 % on a 512 x 512 mesh, 37 % with rows of 8 random entries.
// Sorting needs no LDS but for the products, so that 8 waves fit a SIMD, and no LDS operation waits for another one.  A hash table of
// the row in LDS (a compare-and-swap per product and look, sums there, ranks of the columns by comparing all with all) had room for
// 4 to 7: this kernel 38.8 -> 28.4 us on the mesh, 39.6 -> 24.4 with 65,536 rows of 8 random entries, 12.8 -> 9.3 with 1024 of them,
// 25.6 -> 19.2 for A*P on a 64^3 grid.  With the table's compare-and-swaps and additions requested eight rows of B at a time 45, 56
// and 29: the LDS takes 8 to 12 cycles for each, 30 where eight lanes count in one place, 12 to 17 for an fp64 addition.
// totals: GivenOperands, of each wave: entries, products, and rows of 9 to 16 entries (S_ROW_WIDE) << 1 | whether there are rows of
// other kernels
template <int G, bool kNarrow, typename Operands>
__device__ __forceinline__ void row_small(const SmallArgs &a, const Operands &operands, const uint32_t block, uint3 *totals = nullptr) {
    constexpr int kRows = 64 / G;        // per wave
    constexpr int kAhead = kNarrow ? G / 2 : G;
    extern __shared__ __align__(16) unsigned char small_lds[];
    __shared__ uint32_t s_len[256 / G];
    const int lane = lane_id(), l = lane % G, wave = threadIdx.x >> 6;
    const uint32_t row = block * (256 / G) + threadIdx.x / G;
    const int most = a.shape.products;
    // {key, product} of the row's products, and behind the wave's rows a place for lanes without an element
    uint2 *wave_products = reinterpret_cast<uint2 *>(small_lds + __umul24(wave, a.wave_bytes));
    uint2 *products = wave_products + __umul24(lane / G, most);
    int32_t p = 0, e = 0;
    uint32_t av = 0;
    bool other = false, wide = false;                        // the row is for other kernels; has 9 entries and more
    if (row < a.rows) operands.template list<G>(row, l, most, p, e, av, other, wide);
    // The LDS has room for the row's products: of prepared operands ub says so, and so do the start arrays of those that are
    // canonical; of others the lists are counted here, and a row that has more takes none.
    int len = min(max(e - p, 0), most + 1);
    const int inc16 = row16_inclusive_scan(len);
    int n_products = from_lane<0x15F>(inc16), before = inc16 - len;
    if constexpr (G == 8) {
        const int low = from_lane<0x157>(inc16);
        n_products = lane & 8 ? n_products - low : low;
        before -= lane & 8 ? low : 0;
    }
    if (n_products > most) {
        n_products = len = 0;
        other = other | Operands::kDirect;
    }
    uint32_t wides = 0;
    if constexpr (Operands::kDirect && G == 16) wides = (uint32_t)__popcll(__ballot((l == 0) & wide & (n_products > 0)));
    const uint32_t of_lists = fold_groups<G>(__ballot(len > 0));          // lists that any of the groups has, a bit each
    const int lists = 32 - __builtin_clz(of_lists | 1u);                   // (one, without elements, where there are none)
    // round t: list t, or with narrow lists the lists t * (G / width) ... of the group, and element j of each
    const int width = kNarrow ? a.shape.list_lanes : G, per = kNarrow ? G / width : 1;
    const int j = kNarrow ? l & (width - 1) : l;
    const int rounds = kNarrow ? (lists + per - 1) / per : lists;
    const int from0 = (lane - l + (kNarrow ? l / width : 0)) * 4;          // lane of the round's list, in bytes
    auto of_list = [&](int v, int t) { return __builtin_amdgcn_ds_bpermute(from0 + t * per * 4, v); };
    const int about = before | len << 16;
    const uint32_t idle = (uint32_t)__umul24(kRows - lane / G, most);           // (of the wave, from `products`)
    auto put = [&](const int2 &y, int f, int at, bool on) {
        const float product = __uint_as_float((uint32_t)f) * __uint_as_float((uint32_t)y.y);
        products[on ? (uint32_t)at : idle] = make_uint2((uint32_t)y.x << 8 | (uint32_t)at, __float_as_uint(product));
    };
    // (all requested before any is used; a half, a quarter and a quarter of the rounds there may be, as far as there are any)
    {
        typename Operands::Element x[kAhead];
        int abouts[kAhead];
        auto request = [&](auto from, auto count) {
            constexpr int kFrom = decltype(from)::value, kCount = decltype(count)::value;
            int begin[kCount];
            each_list<kNarrow, G, kFrom>(begin, p, of_list, std::make_integer_sequence<int, kCount>{});
            each_list<kNarrow, G, kFrom>(abouts + kFrom, about, of_list, std::make_integer_sequence<int, kCount>{});
#pragma unroll
            for (int t = 0; t < kCount; ++t) {
                // (rounds of several lists: those past the last one would have lists of other groups)
                if (kNarrow && kFrom + t >= rounds) abouts[kFrom + t] = 0;
                x[kFrom + t] = operands.read((uint32_t)(j < abouts[kFrom + t] >> 16 ? begin[t] + j : 0));
            }
        };
        auto put_round = [&](auto round) {
            constexpr int t = decltype(round)::value;
            put(operands.entry(x[t]), of_round<kNarrow, G, t>((int)av, of_list), (abouts[t] & 0xFFFF) + j, j < abouts[t] >> 16);
        };
        constexpr std::integral_constant<int, 0> k0{};
        constexpr std::integral_constant<int, kAhead / 2> kHalf{};
        constexpr std::integral_constant<int, kAhead / 4> kQuarter{};
        constexpr std::integral_constant<int, kAhead * 3 / 4> kThree{};
        request(k0, kHalf);
        if (rounds > kAhead / 2) request(kHalf, kQuarter);
        if (rounds > kAhead * 3 / 4) request(kThree, kQuarter);
        each_round<0, kAhead / 2>(put_round);
        if (rounds > kAhead / 2) each_round<kAhead / 2, kAhead * 3 / 4>(put_round);
        if (rounds > kAhead * 3 / 4) each_round<kAhead * 3 / 4, kAhead>(put_round);
    }
    // Lists that are longer than their lanes, one round after the other to its end.  The next elements are on their way while some
    // are taken, and rounds without any are left out: chunk by chunk over all rounds, each load waited for, the light rows of graphs
    // of 1000 to 16,000 vertices took 27 to 35 us, 20 to 29 now.
    if (const uint32_t longer = fold_groups<G>(__ballot(len > width))) {
        uint32_t left = longer;                              // rounds that go on, a bit each
        if constexpr (kNarrow) {                             // (per lists to a round)
            left = 0;
            for (int t = 0; t < rounds; ++t) left |= (longer >> (t * per)) & ((1u << per) - 1u) ? 1u << t : 0u;
        }
        int at = 0, end = 0, from = 0, factor = 0;           // of the list's elements, and what is added for their places in B
        typename Operands::Element y;
        auto request = [&] { y = operands.read(at < end ? (uint32_t)(at + from) : 0u); };
        auto next_round = [&] {
            const int t = __builtin_ctz(left);
            const int of = of_list(about, t);
            at = (of & 0xFFFF) + j + width;
            end = (of & 0xFFFF) + (of >> 16);
            from = of_list(p, t) - (of & 0xFFFF);
            factor = of_list((int)av, t);
            left &= left - 1u;
            request();
        };
        next_round();
        for (bool more = true; more;) {
            const typename Operands::Element now = y;
            const int f = factor, place = at;
            const bool on = at < end;
            at += width;
            if (__any(at < end)) request();
            else if (left) next_round();
            else more = false;
            put(operands.entry(now), f, place, on);
        }
    }
    wave_sync();
    int2 *found = a.found + (size_t)(block * 4 + wave) * (kRows * most);
    int n = 0, total = 0;
    auto add_sorted = [&](auto lane_keys) {
        constexpr int R = decltype(lane_keys)::value;
        constexpr uint32_t kNone = ~255u;                    // (place 0: it is read and added to nothing that is wanted)
        uint32_t key[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {                        // (kReadPast: also behind the row's)
            const uint32_t own = products[l * R + r].x;
            key[r] = l * R + r < n_products ? own : kNone;
        }
        sort_group<G, R>(key, l);
        float product[R];
#pragma unroll
        for (int r = 0; r < R; ++r) product[r] = __uint_as_float(products[key[r] & 255u].y);
        // the first and the last of a column's
        bool first[R], last[R];
        const uint32_t previous = from_lane<0x111>(key[R - 1]);
#pragma unroll
        for (int r = 0; r < R; ++r) first[r] = r == 0 ? (l == 0) | ((key[0] ^ previous) > 255u) : (key[r] ^ key[r - 1]) > 255u;
        const uint32_t next = from_lane<0x101>(key[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) last[r] = ((r == R - 1 ? (l == G - 1) | ((key[r] ^ next) > 255u) : first[r == R - 1 ? r : r + 1])) & (key[r] < kNone);
        // what the lanes before have of the column that this one begins with
        double sum = 0;
        bool begun = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sum = (first[r] ? 0.0 : sum) + (double)product[r];
            begun = begun | first[r];
        }
        auto of_before = [&](auto control, double v) {
            const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
            return __builtin_bit_cast(double, (unsigned long long)from_lane<decltype(control)::value>((uint32_t)(bits >> 32)) << 32 |
                                                  from_lane<decltype(control)::value>((uint32_t)bits));
        };
        uint32_t closed = begun ? 1u : 0u;                   // (the first lane of a group always is)
        auto scan_step = [&](auto control) {
            const double other = of_before(control, sum);
            const uint32_t other_closed = from_lane<decltype(control)::value>(closed);
            sum = closed ? sum : sum + other;
            closed |= other_closed;
        };
        scan_step(std::integral_constant<int, 0x111>{});
        scan_step(std::integral_constant<int, 0x112>{});
        scan_step(std::integral_constant<int, 0x114>{});
        if constexpr (G == 16) scan_step(std::integral_constant<int, 0x118>{});
        sum = of_before(std::integral_constant<int, 0x111>{}, sum);
        int own = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) own += last[r] ? 1 : 0;
        const int inc = (int)wave_inclusive_scan((uint32_t)own);
        total = __builtin_amdgcn_readlane(inc, 63);
        n = own;                                             // of the group: pairs, quads, halves of a row, rows
        n += TSP_DPP(0, n, 0xB1, 0xf, true);
        n += TSP_DPP(0, n, 0x4E, 0xf, true);
        n += TSP_DPP(0, n, 0x141, 0xf, true);
        if constexpr (G == 16) n += TSP_DPP(0, n, 0x140, 0xf, true);
        uint32_t to = (uint32_t)(inc - own);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sum = (first[r] ? 0.0 : sum) + (double)product[r];
            if (last[r]) found[to] = make_int2((int)(key[r] >> 8), (int)__float_as_uint((float)sum));
            to += last[r] ? 1u : 0u;
        }
    };
    if (!__any(n_products > G)) add_sorted(std::integral_constant<int, 1>{});
    else if (!__any(n_products > 2 * G)) add_sorted(std::integral_constant<int, 2>{});
    else if (!__any(n_products > 4 * G)) add_sorted(std::integral_constant<int, 4>{});
    else if (!__any(n_products > 8 * G)) add_sorted(std::integral_constant<int, 8>{});
    else if constexpr (G == 16) add_sorted(std::integral_constant<int, 16>{});
    if (lane == 0) a.wave_total[block * 4 + wave] = total;
    if constexpr (Operands::kDirect) {
        // (rows of other kernels count as empty here, and are told of)
        if (l == 0 && row < a.rows) put_for(a.finish, a.row_nnz + row, (int32_t)n);
        const uint32_t of_wave = wave_sum((uint32_t)len), others = __any(other) ? 1u : 0u;
        if (lane == 0) totals[wave] = make_uint3((uint32_t)total, of_wave, wides << 1 | others);
        return;
    }
    if (l == 0) {
        // (rows of other kernels count as empty here)
        if (row < a.rows && !other) put_for(a.finish, a.row_nnz + row, (int32_t)n);
        s_len[threadIdx.x / G] = (uint32_t)n;
    }
    __syncthreads();
    const int64_t g = (int64_t)block * (256 / G / T) + threadIdx.x;
    uint32_t sum_len = 0;
    if (threadIdx.x < 256 / G / T && g * T < a.rows) {
        for (int i = 0; i < T; ++i) sum_len += s_len[threadIdx.x * T + i];
        a.group_len[g] = sum_len;
    }
    if (a.part_len && threadIdx.x < 64) {                       // (one addition per block, whose groups are of one chunk)
        for (int i = 1; i < 256 / G / T; i <<= 1) sum_len += (uint32_t)__shfl_xor((int)sum_len, i, 64);
        if (threadIdx.x == 0) atomicAdd(a.part_len + g / kPartTileRows * kPartStride, sum_len);
    }
    if (a.part_len && block == 0 && threadIdx.x == 0)
        *a.only_small = !(a.d_scalars[S_INVALID] | a.d_scalars[S_ROW_LISTS] | a.d_scalars[S_ROW_LARGE_TASKS]);
}

struct CopyArgs {
    SmallShape shape;
    int64_t rows, waves;
    const int32_t *a_start, *ub;
    const int2 *found;
    const int32_t *wave_total;
    const int64_t *c_row_ptr;
    int32_t *c_col;
    float *c_val;
    const int32_t *live;                 // of k_row_finish, or null
};

// The entries of the small rows into C, a wave per wave of k_row_small: in one piece, since its rows follow one another
// in C, unless a row of another kernel lies between them.
__global__ __launch_bounds__(256) void k_small_copy(const CopyArgs a) {
    if (a.live && !uniform_load(a.live)) return;
    const int lane = lane_id();
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (w >= a.waves) return;
    const int rows = 64 / a.shape.lanes;
    const int64_t r0 = w * rows, r1 = min(r0 + rows, a.rows);
    const int total = uniform_load(a.wave_total + w);
    if (total == 0) return;
    const int64_t first = uniform_load(a.c_row_ptr + r0), last = uniform_load(a.c_row_ptr + r1);
    const int2 *found = a.found + w * (int64_t)(rows * a.shape.products);
    if (last - first == total) {
        int32_t *col = a.c_col + first;
        float *val = a.c_val + first;
        for (int i = lane; i < total; i += 64) {
            const int2 x = found[(unsigned)i];
            col[(unsigned)i] = x.x;
            val[(unsigned)i] = __uint_as_float((uint32_t)x.y);
        }
        return;
    }
    if (!a.ub) return;                       // (k_row_given: no rows of other kernels)
    int from = 0;
    for (int64_t r = r0; r < r1; ++r) {
        const int32_t deg = uniform_load(a.a_start + r + 1) - uniform_load(a.a_start + r), ub = uniform_load(a.ub + r);
        if (deg <= 0 || ub <= 0 || !small_row(deg, ub, a.shape.lanes, a.shape.products)) continue;
        const int64_t to = uniform_load(a.c_row_ptr + r);
        const int n = min((int)(uniform_load(a.c_row_ptr + r + 1) - to), total - from);
        for (int i = lane; i < n; i += 64) {
            const int2 x = found[(unsigned)(from + i)];
            a.c_col[to + i] = x.x;
            a.c_val[to + i] = __uint_as_float((uint32_t)x.y);
        }
        from += n;
    }
}

// The entries of kSideRows rows into C, flat over the threads: `entries_before` them in C, `at` of the block's before this thread's
// row, `own` of the block.
template <int kSideRows>
__device__ __forceinline__ void move_entries(const CopyArgs &c, int64_t side, uint64_t entries_before, uint32_t at, uint64_t own, uint32_t *s_first) {
    const int wave_rows = 64 / c.shape.lanes, waves = kSideRows / wave_rows;
    if ((int)threadIdx.x < kSideRows && threadIdx.x % wave_rows == 0) s_first[threadIdx.x / wave_rows] = at;
    __syncthreads();
    const int64_t wave0 = side * waves;
    const int room = wave_rows * c.shape.products;
    int32_t *col = c.c_col + entries_before;
    float *val = c.c_val + entries_before;
    for (int base = threadIdx.x; base < (int)own; base += 4 * 256) {
        int2 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = (uint32_t)min(base + u * 256, (int)own - 1);
            int w = 0;                                           // the last wave that begins at or before e
#pragma unroll
            for (int d = kSideRows / 8; d > 0; d >>= 1)
                if (w + d < waves && s_first[w + d] <= e) w += d;
            x[u] = c.found[(wave0 + w) * room + (e - s_first[w])];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (base + u * 256 < (int)own) {
                col[base + u * 256] = x[u].x;
                val[base + u * 256] = __uint_as_float((uint32_t)x[u].y);
            }
    }
}

// k_row_finish and k_small_copy at once, for a product launched ahead that is expected to have small rows only: a block takes
// kSideRows rows, adds up the chunks before theirs and the groups before them in it, writes their row_ptr and moves their
// entries, flat over the threads, if what is expected holds.  (On a 512 x 512 mesh the two take 7.4 and 12.4 us one behind the
// other, most of the first in round trips; together 12.0 us, and k_row_small 2 more.  The products: that mesh 69.5 -> 65.7 us,
// 65,536 rows of 8 random entries 65.4 -> 61.4, A*P on a 64^3 grid 65.7 -> 63.8.)
template <int kSideRows>
__global__ __launch_bounds__(256) void k_small_finish(const FinishArgs a, const CopyArgs c, const uint32_t *part_len, const int32_t *only_small) {
    __shared__ uint64_t lds[256 / 64];
    __shared__ PlanTotals totals;
    __shared__ uint32_t s_first[kSideRows / 4];                  // entries of the block before each wave of k_row_small
    // (the first block hands the sizes to the host, which then has the time of this kernel for the next call)
    const bool first = blockIdx.x == 0;
    const int64_t standing = first ? standing_scalar(a.d_scalars) : 0;
    const int64_t row0 = (int64_t)blockIdx.x * kSideRows, row = (int)threadIdx.x < kSideRows ? row0 + threadIdx.x : a.rows;
    const int part = (int)(row0 / kPartRows), parts = (int)((a.rows + kPartRows - 1) / kPartRows);
    const int group0 = part * kPartTileRows, groups = (int)(row0 / T) - group0;            // before the block's, in its part
    uint64_t before = 0, all = 0;
    for (int i = threadIdx.x; i < parts; i += 256) {
        const uint32_t n = part_len[i * kPartStride];
        all += n;
        before += i < part ? n : 0u;
    }
    if ((int)threadIdx.x < groups) before += a.group_len[group0 + threadIdx.x];
    const uint32_t mine = row < a.rows ? (uint32_t)a.row_nnz[row] : 0u;
    if (first) add_plan_sums<false>(a, totals);
    uint64_t entries_before, entries, own;
    (void)block_exclusive_scan64<256>(before, &entries_before, lds);
    (void)block_exclusive_scan64<256>(all, &entries, lds);
    const uint32_t at = (uint32_t)block_exclusive_scan64<256>(mine, &own, lds);
    if (row < a.rows) a.c_row_ptr[row] = (int64_t)(entries_before + at);
    if (first) publish_sizes(a, totals, standing, (int64_t)entries);
    // (No more than this matters where no row is heavy.  Expected::holds also asks whether the heavy rows' accumulator of the last
    // product of these sizes would do for the values: where it would not the host has k_small_copy move the entries once more.)
    // (Also of the block's own end, so that it writes inside C's arrays whatever the sums say.)
    if (!uniform_load(only_small) || (int64_t)entries > a.expected.nnz || (int64_t)(entries_before + own) > a.expected.nnz) return;
    move_entries<kSideRows>(c, blockIdx.x, entries_before, at, own, s_first);
}

// ---- heavy rows -------------------------------------------------------------------------------------------------
// B for the heavy rows, L lanes per row.  For the multiplication: 4 bytes per entry {low 16 bits of the column, fp16
// value}, and where every row of B enters every window of columns.  For the sizing: the columns of a row as words of 16
// {low 16 bits of the word's index, its bits << 16}, at the position of the row's first entry, and where every row enters
// every span of kSpanWindows windows.  (Words of 32 columns in 8 bytes are 0.47 to a product on a power-law graph, weighted by
// use, words of 16 in 4 bytes 0.58: 3.7 and 2.3 bytes.)
struct PackArgs {
    int64_t rows;
    const int32_t *start;
    const int2 *rec;
    uint32_t *pack;                      // (the low five bits of the column inverted: a shift by them brings the column's bit to the top)
    uint32_t *word;
    int32_t *words;                      // per row
    int32_t *table;                      // [rows][windows + 1], or null for one window
    int32_t *span_table;                 // [rows][spans + 1], or null for one span
    int windows, spans, shift;           // a window is 1 << shift columns
    int medium_from;                     // entries from which a row is left to the first blocks
    int lanes;                           // to a row, of the others
    uint32_t blocks;
};
// Bound by latency: a row's trips wait for each other, and the launch for its longest row (25,000 entries of an R-MAT graph
// of scale 18).  So rows of more than pack_short entries are left to the first kLongBlocks blocks.  Each looks through a
// kLongBlocks-th of the rows, works off rows of more than kPackLong with all waves, kTrips trips of every wave to a round, the
// words before a wave's from the others' numbers, and the medium ones by a wave each.  A wave per row throughout was bound by
// the coming and going of 262,144 waves as well.  R-MAT of scale 13/14/16/18: 14.5/24.5/70/209 -> 8.8/11.1/30/139 us (every
// long row by all waves 11.5/16/55/245; medium ones up to 2048 entries 13.5/13.5/33/141; 1024 such blocks 10/13/33/136).
constexpr int kPackThreads = 512;        // of k_heavy_pack
constexpr unsigned kLongBlocks = 256;
constexpr int kPackLong = 1024;
constexpr int pack_short(int L) { return L == 64 ? kPackLong : 128; }
template <int L, bool kLong, int kThreads>
__device__ __forceinline__ void pack_rows(const PackArgs &a, int64_t first_row) {
    constexpr int kTrips = kLong ? 4 : 2, kWaves = kThreads / 64;
    const int l = threadIdx.x % L, lane = lane_id(), span_shift = a.shift + kSpanWindowsLog;
    int64_t row = first_row;
    int32_t s = 0, e = 0, at = 0;
    int32_t *tab = nullptr, *span_tab = nullptr;
    auto take_row = [&](int64_t r) {
        row = r;
        s = e = 0;
        if (row < a.rows) {
            s = a.start[row];
            e = max(s, a.start[row + 1]);
        }
        at = s;
        tab = a.table && row < a.rows ? a.table + row * (a.windows + 1) : nullptr;
        span_tab = a.span_table && row < a.rows ? a.span_table + row * (a.spans + 1) : nullptr;
    };
    int2 xs[kTrips];
    int32_t befores[kTrips];
    auto read = [&](int32_t base) {
#pragma unroll
        for (int u = 0; u < kTrips; ++u) {
            const int32_t k = max(min(base + u * L + l, e - 1), 0);
            xs[u] = a.rec[k];
            befores[u] = a.rec[max(k - 1, 0)].x;
        }
    };
    auto leads = [&](int u, int32_t k) {
        const int32_t before = k > s ? befores[u] : -1;
        return k < e && (l == 0 || before < 0 || (before >> 4) != xs[u].x >> 4);
    };
    auto write = [&](int32_t base) {
#pragma unroll
        for (int u = 0; u < kTrips; ++u) {
            const int32_t k0 = base + u * L, k = k0 + l;
            if (!__any(k0 < e)) break;
            // A word's bits are the difference of the running sum of the bits (all distinct, so that carries cancel) at the two
            // ends of its stretch; a word that goes on in the next trip is listed twice.
            const int2 x = xs[u];
            const int32_t before = k > s ? befores[u] : -1, word = x.x >> 4;
            const uint32_t bit = k < e ? 1u << (x.x & 15) : 0u;
            if (k < e) {
                const _Float16 v = (_Float16)__uint_as_float((uint32_t)x.y);
                a.pack[k] = (((uint32_t)x.x ^ 31u) & 0xFFFFu) | ((uint32_t)__builtin_bit_cast(uint16_t, v) << 16);
                if (tab)
                    for (int w = (before >> a.shift) + 1; w <= (x.x >> a.shift) && w <= a.windows; ++w) tab[w] = k;
            }
            const unsigned long long all = __ballot(leads(u, k)), live = __ballot(k < e);
            const uint32_t sum = wave_inclusive_scan(bit);
            const int start = 63 - __clzll((long long)(all & ((2ull << lane) - 1ull)));
            const uint32_t before_start = (uint32_t)__shfl((int)(sum - bit), max(start, 0), 64);
            const unsigned long long mine = L == 64 ? all : (all >> (lane & ~(L - 1))) & ((1ull << (L & 63)) - 1ull);
            const int32_t place = at + __popcll(mine & ((2ull << l) - 1ull)) - 1;
            if (k < e && (l == L - 1 || !((live >> (lane + 1)) & 1ull) || ((all >> (lane + 1)) & 1ull)))
                a.word[place] = ((uint32_t)word & 0xFFFFu) | (sum - before_start) << 16;
            if (span_tab && k < e)
                for (int w = (before >> span_shift) + 1; w <= (x.x >> span_shift) && w <= a.spans; ++w) span_tab[w] = place;
            at += __popcll(mine);
        }
    };
    auto close_row = [&]() {
        if (row < a.rows && l == 0) a.words[row] = at - s;
        const int32_t last_column = e > s && (tab || span_tab) ? a.rec[e - 1].x : -1;
        if (tab)
            for (int w = (last_column < 0 ? -1 : min(last_column >> a.shift, a.windows - 1)) + 1 + l; w <= a.windows; w += L) tab[w] = e;
        if (span_tab)
            for (int w = (last_column < 0 ? -1 : min(last_column >> span_shift, a.spans - 1)) + 1 + l; w <= a.spans; w += L) span_tab[w] = at;
    };

    if constexpr (!kLong) {
        take_row(first_row);
        if (e - s > pack_short(L)) take_row(a.rows);         // (none)
        for (int32_t base = s; __any(base < e); base += L * kTrips) {
            read(base);
            write(base);
        }
        close_row();
    } else {
        __shared__ int64_t s_long[kThreads];
        __shared__ int32_t s_words[2][kWaves], s_n[2];
        const int wave = threadIdx.x >> 6;
        int round = 0;
        // (neighbours are looked at by different blocks, and those of the next kLongBlocks rows by others again: in graphs the
        // long rows lie together or at regular distances)
        for (int64_t group = 0; group * kLongBlocks < a.rows; group += kThreads) {
            const int64_t g = group + threadIdx.x, r = g * kLongBlocks + (blockIdx.x + 101 * g) % kLongBlocks;
            if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
            __syncthreads();
            const int32_t len = r < a.rows ? a.start[r + 1] - a.start[r] : 0;
            if (len > kPackLong) s_long[atomicAdd(&s_n[0], 1)] = r;
            else if (len >= a.medium_from) s_long[kThreads - 1 - atomicAdd(&s_n[1], 1)] = r;
            __syncthreads();
            const int n_long = s_n[0], n_medium = s_n[1];
            for (int q = 0; q < n_long; ++q) {
                take_row(s_long[q]);
                for (int32_t first = s; first < e; first += kWaves * kTrips * 64, round ^= 1) {
                    const int32_t base = first + wave * kTrips * 64;
                    read(base);
                    int n = 0;
#pragma unroll
                    for (int u = 0; u < kTrips; ++u) n += __popcll(__ballot(leads(u, base + u * 64 + l)));
                    if (lane == 0) s_words[round][wave] = n;
                    __syncthreads();         // (the other half is written next: nobody is more than a barrier ahead)
                    const int32_t of = lane < kWaves ? s_words[round][lane] : 0;
                    const int32_t inc = (int32_t)wave_inclusive_scan((uint32_t)of), begun = at;
                    at = begun + __builtin_amdgcn_readlane(inc - of, wave);
                    write(base);
                    at = begun + __builtin_amdgcn_readlane(inc, 63);
                }
                if (wave == 0) close_row();
            }
            for (int q = wave; q < n_medium; q += kWaves) {
                take_row(s_long[kThreads - 1 - q]);
                for (int32_t base = s; base < e; base += kTrips * 64) {
                    read(base);
                    write(base);
                }
                close_row();
            }
            __syncthreads();
        }
    }
}
template <int kThreads>
__device__ __forceinline__ void pack_block(const PackArgs &a, uint32_t block) {
    if (block < kLongBlocks) pack_rows<64, true, kThreads>(a, 0);
    else if (a.lanes == 16) pack_rows<16, false, kThreads>(a, ((int64_t)(block - kLongBlocks) * kThreads + threadIdx.x) / 16);
    else pack_rows<64, false, kThreads>(a, ((int64_t)(block - kLongBlocks) * kThreads + threadIdx.x) / 64);
}
__global__ __launch_bounds__(kPackThreads) void k_heavy_pack(const PackArgs a) { pack_block<kPackThreads>(a, blockIdx.x); }
struct NoPack {};

// The blocks that sum come first or last.  Before them those of k_heavy_pack (Pack) where B has up to kPackRows rows: they need
// nothing of the small rows, and both are bound by latency.  The two kernels, one behind the other and at once: 4099 rows of 37
// entries times as many 15.5 and 11.6 us, R-MAT of scale 14 39 and 35; products of scale 11 60 and 54, of scale 16, with 12 entries
// per row, 945 and 950; of scale 18, which fills the chip either way and has fewer waves here, the two 434 and 476.
constexpr int64_t kPackRows = 1 << 15;
template <int G, bool kNarrow, typename Pack = NoPack>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_row_small(const SmallArgs a, const PreparedOperands operands, const SumArgs sums, const FinishArgs fin, const Pack pack) {
    __shared__ int s_last;
    uint32_t block = blockIdx.x, blocks = gridDim.x;
    if constexpr (!std::is_same<Pack, NoPack>::value) {
        if (block < pack.blocks) {
            pack_block<256>(pack, block);
            return;
        }
        block -= pack.blocks;
        blocks -= pack.blocks;
    }
    const int sum_block = (int)block - (a.sums_first ? 0 : (int)blocks - a.sum_blocks);
    if (sum_block >= 0 && sum_block < a.sum_blocks) sum_tile_rows(sums, sum_block, a.sum_blocks, a.finish);
    else row_small<G, kNarrow>(a, operands, block - (a.sums_first ? (uint32_t)a.sum_blocks : 0u));
    if (!a.finish) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // what this wave has left for the last block has arrived
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = atomicAdd(reinterpret_cast<unsigned long long *>(fin.d_scalars + S_ROW_ARRIVED), 1ull) == blocks - 1;
    __syncthreads();
    if (s_last) row_finish<true>(fin, 0, 1);
}

// ---- small rows straight from the operands ------------------------------------------------------------------------
// A product of sizes whose last product had small rows only needs no records of its entries, and no list of other rows.  One launch
// has blocks that look the operands over (validation, tiles), blocks that take rows as the caller gave them (GivenOperands), and
// blocks that add up the pairs of tiles; the last of all hands the sizes to the host, which has the time of the next launch for the
// next call.  That one makes row_ptr and moves the entries into C (k_given_finish); for products of one chunk of rows the last block
// makes row_ptr, and k_small_copy moves them.  Where a row turns out to be for other kernels the product is started again with
// k_row_prepare.
// Bound by vector instructions where there are many rows (70 % of the time on the 512 x 512 mesh, with 4.8 waves per SIMD that wait for
// 42 % of theirs), and by round trips where there are few or a launch begins and ends (37 x 37: waves wait for 74 %); so fewer launches,
// with more of different kinds in each.  k_row_prepare, k_row_small and k_small_finish, one behind the other, against these
// two: a 512 x 512 mesh 16.1 + 28.4 + 12.1 us and 36.0 + 12.7, 65,536 rows of 8 random entries 10.8 + 24.4 + 12.3 and 29.6 + 12.8,
// A*P on a 64^3 grid 25.6 + 19.2 + 6.7 and 30.6 + 7.4; the products 56.4 -> 45.5, 47.3 -> 40.5, 58.5 -> 39.1, a 37 x 37 mesh 26.6 ->
// 17.9, 1024 rows of 8 entries 27.0 -> 19.2.  The pairs of tiles from lists of A's tiles in every tile-row take three round trips, from
// A's tiles in every tile column one (the choice: rowwise_given): 37 x 37 mesh 15.5 -> 9.7 us of the launch, 135 x 135 14.8 -> 13.0.  Without the pairs of tiles 33.6, 24.3 and 28.3 us, but added up by blocks of the second
// launch they hand the sizes over so late that the GPU waits for the next call (58.3, 49.1, 53.6).  Blocks that count themselves with
// an addition whose result they wait for, 38.4, 33.6 and 38.4 us; one block that looks at the counters needs no such wait.
template <typename RP>
struct TileArgs {                        // of an operand
    const RP *row_ptr;
    const int32_t *col;
    int64_t rows, cols, nnz;
    int bitmap_words;
    int32_t *ntiles;                     // of every tile-row
    // Of A: per tile column, how many tile-rows have a tile in it; or of every tile-row the first entry and, from there on, the columns of
    // its tiles in any order (null: not wanted)
    uint32_t *counts;
    int32_t *first, *tile_col;
};

// A wave for `per_wave` (1 or 4) tile-rows, two entries per lane in flight and the next tile-row's first ones: k_row_prepare without
// what is kept of the entries.  Other blocks of the launch read what it leaves.  The number of tiles of the wave's.
template <bool kCounts, typename RP>
__device__ __forceinline__ int32_t count_tiles(const TileArgs<RP> &a, uint32_t block, int per_wave, bool validate, int64_t *d_scalars) {
    extern __shared__ __align__(16) unsigned char small_lds[];
    __shared__ uint32_t s_starts[4][4];  // of the entries of a trip, those that begin a row
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t *bitmap = reinterpret_cast<uint32_t *>(small_lds) + wave * a.bitmap_words, *starts = s_starts[wave];
    const int64_t I0 = ((int64_t)block * 4 + wave) * per_wave;
    if (I0 * T >= a.rows) return 0;
    // lane 16 t + r: row r of tile-row t, and of all lanes the row behind the last
    const int64_t i = min(I0 * T + lane, a.rows), behind = min((I0 + per_wave) * T, a.rows);
    auto clamped = [&](RP raw) { return (int32_t)min(max(raw, (RP)0), (RP)a.nnz); };
    const RP raw = a.row_ptr[i], raw_behind = a.row_ptr[behind];
    const int32_t q = clamped(raw), end = clamped(raw_behind);
    int32_t p = q;
    p = max(p, TSP_DPP(p, p, 0x111, 0xf, false));
    p = max(p, TSP_DPP(p, p, 0x112, 0xf, false));
    p = max(p, TSP_DPP(p, p, 0x114, 0xf, false));
    p = max(p, TSP_DPP(p, p, 0x118, 0xf, false));
    bool bad = lane < per_wave * T && (raw != (RP)p || (i == 0 && raw != 0) || (i == a.rows && raw != (RP)a.nnz));
    bad = bad | (raw_behind != (RP)end) | (behind == a.rows && raw_behind != (RP)a.nnz);
    auto begin_of = [&](int t) { return t < per_wave ? __builtin_amdgcn_readlane(q, t * T) : end; };
    int32_t all = 0;
    int32_t next[2];                     // columns of the tile-row's first entries
    auto request = [&](int32_t from, int32_t to) {
#pragma unroll
        for (int u = 0; u < 2; ++u) next[u] = a.col[max(min(from + u * 64 + lane, to - 1), 0)];
    };
    auto end_of = [&](int t) { return max(__builtin_amdgcn_readlane(p, t * T + T - 1), begin_of(t + 1)); };
    request(begin_of(0), end_of(0));
    for (int t = 0; t < per_wave && (I0 + t) * T < a.rows; ++t) {
        const int32_t e0 = begin_of(t), e1 = end_of(t);
        // (what follows a tile-row is no less than its end, or the operand is not canonical)
        bad = bad | (e1 != begin_of(t + 1));
        for (int w = lane; w < a.bitmap_words / 4; w += 64) reinterpret_cast<uint4 *>(bitmap)[w] = make_uint4(0, 0, 0, 0);
        int32_t c[2] = {next[0], next[1]};
        if (t + 1 < per_wave) request(begin_of(t + 1), end_of(t + 1));
        int32_t listed = 0, before = 0;  // column of the entry before the trip
        for (int32_t base = e0; base < e1; base += 128) {
            if (base > e0)
#pragma unroll
                for (int u = 0; u < 2; ++u) c[u] = a.col[min(base + u * 64 + lane, e1 - 1)];
            if (lane < 4) starts[lane] = 0;
            wave_sync();
            if (lane / T == t && (uint32_t)(p - base) < 128u) atomicOr(&starts[(p - base) >> 5], 1u << ((p - base) & 31));
            wave_sync();
            uint32_t begins[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) begins[u] = starts[2 * u + (lane >> 5)] >> (lane & 31);
            int32_t prev[2];
            prev[0] = TSP_DPP(before, c[0], 0x138, 0xf, false);            // wave_shr:1
            prev[1] = TSP_DPP(__builtin_amdgcn_readlane(c[0], 63), c[1], 0x138, 0xf, false);
            before = __builtin_amdgcn_readlane(c[1], 63);
            uint32_t had[2];
            bool first[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int32_t k = base + u * 64 + lane;
                const bool on = k < e1, outside = (uint32_t)c[u] >= (uint64_t)a.cols;
                bad = bad | (on & (outside | (!(begins[u] & 1u) & (prev[u] >= c[u]))));
                if (outside) c[u] = 0;
                // (of the entries of a tile one behind the other, also over the end of a row, the first)
                first[u] = on & ((k == e0) | ((prev[u] >> 4) != (c[u] >> 4)));
                had[u] = first[u] ? atomicOr(&bitmap[c[u] >> 9], 1u << ((c[u] >> 4) & 31)) : 0u;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                first[u] = first[u] & !((had[u] >> ((c[u] >> 4) & 31)) & 1u);
                const unsigned long long firsts = __ballot(first[u]);
                if (kCounts && first[u] && a.counts) atomicAdd(a.counts + (c[u] >> 4), 1u);
                if (!kCounts && first[u] && a.tile_col) put_for(true, a.tile_col + e0 + listed + __popcll(firsts & ((1ull << lane) - 1ull)), c[u] >> 4);
                listed += __popcll(firsts);
            }
        }
        if (lane == 0) {
            if (!kCounts && a.first) put_for(true, a.first + I0 + t, e0);
            put_for(true, a.ntiles + I0 + t, listed);
        }
        all += listed;
        wave_sync();
    }
    if (bad && validate) put_for(true, d_scalars + S_INVALID, (int64_t)1);
    return all;
}

// Blocks of a launch that count themselves, in groups of kArriveGroup, with what they have to add up: a counter per group, zero
// before and after.  (An addition to one counter is 9 ns; 8192 of them would outlast the launch.)  Blocks in the upper 8 bits, below
// them what the blocks add up.
constexpr int kArriveGroup = 64;
constexpr int kArriveShift = 56;
constexpr unsigned long long kArriveSum = (1ull << kArriveShift) - 1ull;
// ... of rows: entries, products, blocks with rows of other kernels, rows of 9 to 16 entries
struct GroupOfRows {
    static constexpr int kProducts = 18, kOthers = 36, kWide = 43;
    static constexpr unsigned long long pack(uint32_t entries, uint32_t products, uint32_t others, uint32_t wide) {
        return 1ull << kArriveShift | (unsigned long long)wide << kWide | (unsigned long long)others << kOthers | (unsigned long long)products << kProducts | entries;
    }
    static_assert(kArriveGroup * 16 * 192 < 1 << kProducts && kArriveGroup * 32 * 96 < 1 << kProducts && kOthers - kProducts == kProducts, "sums over a group");
    static_assert(kArriveGroup < 1 << (kWide - kOthers) && kArriveGroup * 16 < 1 << (kArriveShift - kWide), "(8 lanes to a row have no rows of 9 entries)");
    uint32_t entries, products, others, wide;
    __device__ explicit GroupOfRows(unsigned long long sum)
        : entries((uint32_t)sum & ((1u << kProducts) - 1u)), products((uint32_t)(sum >> kProducts) & ((1u << kProducts) - 1u)),
          others((uint32_t)(sum >> kOthers) & ((1u << (kWide - kOthers)) - 1u)), wide((uint32_t)(sum >> kWide) & ((1u << (kArriveShift - kWide)) - 1u)) {}
};
__host__ __device__ constexpr uint32_t arrive_groups(uint32_t blocks) { return (blocks + kArriveGroup - 1) / kArriveGroup; }
__device__ __forceinline__ uint32_t arrive_blocks(uint32_t group, uint32_t blocks) { return min(blocks - group * kArriveGroup, (uint32_t)kArriveGroup); }
// The blocks of a launch are dispatched in order, so those before a block that waits run or are done.  Waits are bounded all the same:
// so many looks (0: none that counts), a microsecond each, and the host starts the product again.
constexpr unsigned kArriveSpins = 1u << 18;
template <typename X, typename Done>
__device__ __forceinline__ X wait_for(const X *p, unsigned looks, Done done, bool *failed) {
    X v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned spins = 0;
    while (spins < looks && !done(v)) {
        if (++spins < looks) __builtin_amdgcn_s_sleep(2);
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    *failed = *failed | (spins >= looks);
    return v;
}
__device__ __forceinline__ unsigned long long add_scalar(int64_t *d_scalars, int slot, unsigned long long v) {
    return atomicAdd(reinterpret_cast<unsigned long long *>(d_scalars + slot), v);
}

struct GivenPublishArgs {
    int64_t rows, room;                  // room: entries that the arrays of C hold
    int64_t *c_row_ptr;
    int64_t *d_scalars, *h_scalars_dev;
    int64_t publish_tag;
    int32_t *live;                       // of k_small_copy, or null: whether it may run
    int same;                            // A and B are one matrix
};
// publish_scalars by one wave; the numbers of tiles, `candidates` and `failed` beyond what stands in the scalar block
__device__ __forceinline__ void publish_given(const GivenPublishArgs &a, int64_t entries, int64_t products, int64_t others, int64_t wide, int64_t tiles_a,
                                              int64_t tiles_b, int64_t candidates, int64_t failed) {
    const int lane = lane_id();
    int64_t v = 0;
    if (lane < kScalars) v = __hip_atomic_load(a.d_scalars + (a.same && lane == S_TILES_B ? (int)S_TILES_A : lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = lane == S_C_NNZ ? entries : lane == S_ROW_PRODUCTS ? products : lane == S_ROW_HEAVY ? others : lane == S_ROW_WIDE ? wide : lane == S_CANDIDATES ? v + candidates : lane == S_INTERNAL ? v + failed : v;
    v += lane == S_TILES_A || (a.same && lane == S_TILES_B) ? tiles_a : lane == S_TILES_B ? tiles_b : 0;
    const bool invalid = __any((lane == S_INVALID || lane == S_INTERNAL) && v != 0);
    if (lane < kScalars) {
        const uint64_t slot = (publish_tag16(a.publish_tag) << kPublishTagShift) | ((uint64_t)v & ((1ull << kPublishTagShift) - 1u));
        __hip_atomic_store(&a.h_scalars_dev[lane], (int64_t)slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        a.d_scalars[lane] = 0;
    }
    if (lane == 0) {
        a.c_row_ptr[a.rows] = entries;
        if (a.live) *a.live = !invalid && !others && entries <= a.room;
    }
}

// B's tile-rows, of a product of one chunk of rows, up to which the last block has the pairs of tiles itself; otherwise other blocks do.
constexpr int kPairsByOne = 4096;
template <typename RP, typename VT>
struct GivenArgs {
    SmallArgs small;
    GivenOperands<RP, VT> operands;
    TileArgs<RP> a, b;
    int64_t a_tile_rows, b_tile_rows;
    const int32_t *b_ntiles;
    // blocks of the launch: tiles of A, of B (none if it is A), rows, with those for the pairs of tiles (none for one chunk of rows)
    // among them, and one that waits for all others
    uint32_t a_blocks, b_blocks, row_blocks, pair_blocks;
    int per_wave;                        // tile-rows
    int validate;
    unsigned looks;                      // of a block that waits
    unsigned long long *counters;        // of groups of blocks: tiles of A, of B, rows
    GivenPublishArgs publish;
};

// The pairs of tiles: of every column A's tiles times the tiles of B's tile-row, 256 at a time, every `blocks`-th of those; the counts are
// zero behind it.  The thread's share.
template <typename RP, typename VT>
__device__ __forceinline__ unsigned long long count_pairs(const GivenArgs<RP, VT> &a, uint32_t block, uint32_t blocks) {
    unsigned long long pairs = 0;
    const int64_t step = (int64_t)blocks * 256;
    for (int64_t K0 = (int64_t)block * 256 + threadIdx.x; K0 < a.b_tile_rows; K0 += 4 * step) {
        uint32_t of_a[4], of_b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t K = K0 + u * step;
            of_a[u] = K < a.b_tile_rows ? get_shared<true>(a.a.counts + K) : 0u;
            of_b[u] = K < a.b_tile_rows ? (uint32_t)get_shared<true>(a.b_ntiles + K) : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            pairs += (unsigned long long)of_a[u] * of_b[u];
            if (K0 + u * step < a.b_tile_rows) put_for(true, a.a.counts + K0 + u * step, 0u);
        }
    }
    return pairs;
}
// The pairs of tiles of 16 tile-rows of A at a time, every `blocks`-th 16: 16 lanes to a tile-row, four tile-rows and of each 64
// tiles in flight.  The thread's share.
template <typename RP, typename VT>
__device__ __forceinline__ unsigned long long count_listed_pairs(const GivenArgs<RP, VT> &a, uint32_t block, uint32_t blocks) {
    const int r = threadIdx.x & 15;
    unsigned long long pairs = 0;
    for (int64_t base = (int64_t)block * 16 + (threadIdx.x >> 4); base < a.a_tile_rows; base += (int64_t)blocks * 64) {
        int32_t first[4], n[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t I = base + (int64_t)blocks * 16 * u;
            first[u] = n[u] = 0;
            if (I < a.a_tile_rows) {
                first[u] = get_shared<true>(a.a.first + I);
                n[u] = get_shared<true>(a.a.ntiles + I);
            }
        }
        for (int32_t j = r; __any(j < max(max(n[0], n[1]), max(n[2], n[3]))); j += 64) {
            int32_t K[4][4], of_b[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) K[u][v] = j + 16 * v < n[u] ? get_shared<true>(a.a.tile_col + first[u] + j + 16 * v) : INT32_MAX;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) of_b[u][v] = K[u][v] < a.b_tile_rows ? get_shared<true>(a.b_ntiles + K[u][v]) : 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) pairs += (uint32_t)of_b[u][v];
        }
    }
    return pairs;
}
// The sum over the block, in its first thread
__device__ __forceinline__ unsigned long long add_threads(unsigned long long v, unsigned long long (&s_sum)[4]) {
    const unsigned long long of_wave = wave_inclusive_scan64(v);
    __syncthreads();
    if (lane_id() == 63) s_sum[threadIdx.x >> 6] = of_wave;
    __syncthreads();
    return s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

template <int G, bool kNarrow, bool kCounts, typename RP, typename VT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_row_given(const GivenArgs<RP, VT> a) {
    __shared__ uint3 s_totals[4];
    __shared__ unsigned long long s_sum[4];
    const uint32_t tile_blocks = a.a_blocks + a.b_blocks, tile_groups = arrive_groups(a.a_blocks) + arrive_groups(a.b_blocks), row_groups = arrive_groups(a.row_blocks);
    const bool one_chunk = a.small.finish;
    int64_t *d_scalars = a.publish.d_scalars;
    if (blockIdx.x < tile_blocks) {
        const bool of_b = blockIdx.x >= a.a_blocks;
        const uint32_t block = blockIdx.x - (of_b ? a.a_blocks : 0u), blocks = of_b ? a.b_blocks : a.a_blocks;
        const int32_t tiles = count_tiles<kCounts>(of_b ? a.b : a.a, block, a.per_wave, a.validate, d_scalars);
        if (lane_id() == 0) s_totals[threadIdx.x >> 6].x = (uint32_t)tiles;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // what this wave has left for other blocks has arrived
        __syncthreads();
        if (threadIdx.x > 0) return;
        unsigned long long *counter = a.counters + ((of_b ? arrive_groups(a.a_blocks) : 0u) + block / kArriveGroup) * kArriveStride;
        const unsigned long long mine = (unsigned long long)s_totals[0].x + s_totals[1].x + s_totals[2].x + s_totals[3].x;
        if (kCounts && !a.pair_blocks) {                       // (the last block looks at the counters itself)
            atomicAdd(counter, mine + (1ull << kArriveShift));
            return;
        }
        // the last of its group tells the others
        const unsigned long long had = atomicAdd(counter, mine + (1ull << kArriveShift));
        if ((had >> kArriveShift) + 1 != arrive_blocks(block / kArriveGroup, blocks)) return;
        __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        (void)add_scalar(d_scalars, of_b ? S_TILES_B : S_TILES_A, (had & kArriveSum) + mine);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        (void)add_scalar(d_scalars, S_GIVEN_ARRIVED, 1);
        return;
    }
    // (the pairs after half of the rows: the tiles are done by then, and their round trips pass beside the other half)
    const uint32_t at = blockIdx.x - tile_blocks, half = a.row_blocks / 2;
    if (at < half || (at >= half + a.pair_blocks && at < a.row_blocks + a.pair_blocks)) {
        const uint32_t block = at < half ? at : at - a.pair_blocks;
        row_small<G, kNarrow>(a.small, a.operands, block, s_totals);
        if (one_chunk) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // (the last block reads row_nnz)
        __syncthreads();
        if (threadIdx.x > 0) return;
        uint32_t entries = 0, products = 0, others = 0, wide = 0;
        for (int w = 0; w < 4; ++w) {
            entries += s_totals[w].x;
            products += s_totals[w].y;
            others |= s_totals[w].z & 1u;
            wide += s_totals[w].z >> 1;
        }
        if (!one_chunk) a.small.block_len[block] = entries;
        atomicAdd(a.counters + (tile_groups + block / kArriveGroup) * kArriveStride, GroupOfRows::pack(entries, products, others, wide));
        return;
    }
    const bool last = at == a.row_blocks + a.pair_blocks;
    bool failed = false;
    unsigned long long pairs = 0, tiles_a = 0, tiles_b = 0;
    if (!last) {
        if (threadIdx.x == 0) (void)wait_for(d_scalars + S_GIVEN_ARRIVED, a.looks, [&](int64_t v) { return v == (int64_t)tile_groups; }, &failed);
        // (lists that are not there yet could lead anywhere)
        if (!__syncthreads_or(failed))
            pairs = add_threads(kCounts ? count_pairs(a, at - half, a.pair_blocks) : count_listed_pairs(a, at - half, a.pair_blocks), s_sum);
        if (threadIdx.x > 0) return;
        (void)add_scalar(d_scalars, S_CANDIDATES, pairs);
        if (failed) (void)add_scalar(d_scalars, S_INTERNAL, 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        (void)add_scalar(d_scalars, S_ROW_ARRIVED, 1);
        return;
    }
    if (kCounts && !a.pair_blocks) {
        static_assert(arrive_groups(kChunkTileRows / 4) + arrive_groups(kPairsByOne / 4) <= 64, "the first wave has them all");
        const uint32_t a_groups = arrive_groups(a.a_blocks);
        if (threadIdx.x < 64) {
            unsigned long long tiles = 0;
            if (threadIdx.x < tile_groups) {
                const bool of_b = threadIdx.x >= a_groups;
                unsigned long long *counter = a.counters + threadIdx.x * kArriveStride;
                const unsigned long long want = arrive_blocks(of_b ? threadIdx.x - a_groups : threadIdx.x, of_b ? a.b_blocks : a.a_blocks);
                tiles = wait_for(counter, a.looks, [&](unsigned long long v) { return (v >> kArriveShift) == want; }, &failed) & kArriveSum;
                __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            tiles_a = wave_sum(threadIdx.x < a_groups ? (uint32_t)tiles : 0u);
            tiles_b = wave_sum(threadIdx.x < a_groups ? 0u : (uint32_t)tiles);
        }
        __syncthreads();
        pairs = add_threads(count_pairs(a, 0u, 1u), s_sum);
    }
    // the last block: the groups of blocks of rows, and the other blocks of pairs
    unsigned long long sum = 0;
    if (threadIdx.x < row_groups) {
        unsigned long long *counter = a.counters + (tile_groups + threadIdx.x) * kArriveStride;
        sum = wait_for(counter, a.looks, [&](unsigned long long v) { return (v >> kArriveShift) == arrive_blocks(threadIdx.x, a.row_blocks); }, &failed);
        __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x == 0 && a.pair_blocks) (void)wait_for(d_scalars + S_ROW_ARRIVED, a.looks, [&](int64_t v) { return v == (int64_t)a.pair_blocks; }, &failed);
    const GroupOfRows group(sum);
    const uint32_t of_wave[4] = {wave_sum(group.entries), wave_sum(group.products), wave_sum(group.others), wave_sum(group.wide)};
    const bool any_failed = __any(failed);
    // (of a wave's 64 groups at most 2^12 blocks and 2^16 rows)
    if (lane_id() == 0) s_totals[threadIdx.x >> 6] = make_uint3(of_wave[0], of_wave[1], of_wave[2] << 18 | of_wave[3] | (any_failed ? 1u << 31 : 0u));
    __syncthreads();
    if (threadIdx.x < 64) {
        int64_t entries = 0, products = 0, others = 0, wide = 0, failures = 0;
        for (int w = 0; w < 4; ++w) {
            entries += s_totals[w].x;
            products += s_totals[w].y;
            others += (s_totals[w].z & 0x7FFFFFFFu) >> 18;
            wide += s_totals[w].z & ((1u << 18) - 1u);
            failures += s_totals[w].z >> 31;
        }
        publish_given(a.publish, entries, products, others, wide, (int64_t)tiles_a, (int64_t)tiles_b, (int64_t)pairs, failures);
    }
    if (!one_chunk) return;
    // row_ptr of one chunk of rows
    __shared__ uint64_t lds[256 / 64];
    constexpr int kItems = kChunkRows / 256;
    const int base = (int)threadIdx.x * kItems;
    uint32_t x[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) x[i] = base + i < a.small.rows ? (uint32_t)get_shared<true>(a.small.row_nnz + base + i) : 0u;
    uint64_t of_thread = 0, total;
#pragma unroll
    for (int i = 0; i < kItems; ++i) of_thread += x[i];
    uint64_t run = block_exclusive_scan64<256>(of_thread, &total, lds);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (base + i < a.small.rows) a.publish.c_row_ptr[base + i] = (int64_t)run;
        run += x[i];
    }
}

// Behind k_row_given, kSideRows rows to a block: their row_ptr, and their entries into C.  The entries before theirs from the numbers
// of the blocks of rows.
template <int kSideRows>
__global__ __launch_bounds__(256) void k_given_finish(const CopyArgs c, int64_t *c_row_ptr, const int32_t *row_nnz, const uint32_t *block_len, int64_t room) {
    __shared__ uint64_t lds[256 / 64];
    __shared__ uint32_t s_first[kSideRows / 4];                  // entries of the block before each wave of k_row_given
    const int64_t row0 = (int64_t)blockIdx.x * kSideRows, row = (int)threadIdx.x < kSideRows ? row0 + threadIdx.x : c.rows;
    const int blocks_before = (int)(row0 * c.shape.lanes / 256);
    const uint32_t mine = row < c.rows ? (uint32_t)row_nnz[row] : 0u;
    uint64_t before = 0;
    const uint4 *len4 = reinterpret_cast<const uint4 *>(block_len);
    for (int i0 = threadIdx.x; i0 * 4 < blocks_before; i0 += 8 * 256) {
        uint4 len[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) len[u] = len4[min(i0 + u * 256, (blocks_before - 1) / 4)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int left = blocks_before - (i0 + u * 256) * 4;
            before += left > 0 ? len[u].x : 0u;
            before += left > 1 ? len[u].y : 0u;
            before += left > 2 ? len[u].z : 0u;
            before += left > 3 ? len[u].w : 0u;
        }
    }
    uint64_t entries_before, own;
    (void)block_exclusive_scan64<256>(before, &entries_before, lds);
    const uint32_t at = (uint32_t)block_exclusive_scan64<256>(mine, &own, lds);
    if (row < c.rows) c_row_ptr[row] = (int64_t)(entries_before + at);
    if ((int64_t)(entries_before + own) > room) return;         // (the host has k_small_copy move all entries once more)
    move_entries<kSideRows>(c, blockIdx.x, entries_before, at, own, s_first);
}

// 64 pieces of up to 16 elements of B, four to a step: lane 16 q + t describes piece 4 t + q by the byte offset of its first
// element and `about`, its number of elements << 16 | 16 bits of its own, and step t hands both to the 16 lanes that read the
// piece (row_newbcast: an operand modifier of the instructions that use them; reading descriptions back from LDS cost an LDS
// instruction per step).  Up to eight steps' elements are requested together.  use(x, about, l) gets the elements of up to
// four steps, what describes them, and this lane's place in the piece: lanes past the end of a piece have other elements, up
// to 15 past the segment.
template <int kFirst, typename X, typename Use, int... kStep>
__device__ __forceinline__ void use_steps(int about, const X *x, Use &use, std::integer_sequence<int, kStep...>) {
    const X y[] = {x[kStep]...};
    const uint32_t d[] = {(uint32_t)TSP_DPP(0, about, 0x150 + kFirst + kStep, 0xf, true)...};
    use(y, d, threadIdx.x % 16u);
}
template <int kFirst, typename X, typename Use, int... kStep>
__device__ __forceinline__ void read_steps(int byte, int about, const X *from, Use &use, std::integer_sequence<int, kStep...>) {
    constexpr int kCount = sizeof...(kStep), kFour = kCount < 4 ? kCount : 4;
    const uint32_t my_byte = threadIdx.x % 16u * (uint32_t)sizeof(X);
    const X x[] = {*reinterpret_cast<const X *>(reinterpret_cast<const char *>(from) +
                                                ((uint32_t)TSP_DPP(0, byte, 0x150 + kFirst + kStep, 0xf, true) + my_byte))...};
    // (four at a time: eight want more registers than there are)
    use_steps<kFirst>(about, x, use, std::make_integer_sequence<int, kFour>{});
    if constexpr (kCount > 4) use_steps<kFirst + 4>(about, x + 4, use, std::make_integer_sequence<int, kCount - 4>{});
}
template <typename X, typename Use>
__device__ __forceinline__ void read_pieces(int byte, int about, int pieces, const X *from, Use &use) {
    const int steps = (pieces + 3) / 4;
    auto batch = [&](auto first, int n) {
        constexpr int kFirst = decltype(first)::value;
        if (n > 4) read_steps<kFirst>(byte, about, from, use, std::make_integer_sequence<int, 8>{});
        else if (n > 2) read_steps<kFirst>(byte, about, from, use, std::make_integer_sequence<int, 4>{});
        else if (n == 2) read_steps<kFirst>(byte, about, from, use, std::make_integer_sequence<int, 2>{});
        else if (n == 1) read_steps<kFirst>(byte, about, from, use, std::make_integer_sequence<int, 1>{});
    };
    batch(std::integral_constant<int, 0>{}, steps);
    batch(std::integral_constant<int, 8>{}, steps - 8);
}

// The segments of B behind up to 64 entries of A, one per lane (first element, length, 16 bits of its own), as pieces of G
// elements, 64 / G pieces to a step of the wave.  The lanes describe 64 pieces at a time: the segment that a piece lies in
// from a running maximum over the marks the segments leave at their first pieces.
template <int G, typename X, typename Use>
__device__ __forceinline__ void stream_pieces(int p, int len, uint32_t own, const X *from, uint32_t *mark, Use use) {
    const int lane = lane_id();
    const int count = len > 0 ? (len + G - 1) / G : 0;
    const int inc = (int)wave_inclusive_scan((uint32_t)count), first = inc - count;
    const int total = __builtin_amdgcn_readlane(inc, 63);
    const int mine = G == 16 ? 4 * (lane % 16) + lane / 16 : lane;             // the piece this lane describes (read_pieces)
    int carry = 0;
    for (int j0 = 0; j0 < total; j0 += 64) {
        mark[lane] = 0;
        wave_sync();
        if (count > 0 && (uint32_t)(first - j0) < 64u) mark[first - j0] = (uint32_t)lane + 1u;
        wave_sync();
        int m = max((int)mark[lane], lane == 0 ? carry : 0);
        m = max(m, TSP_DPP(m, m, 0x111, 0xf, false));
        m = max(m, TSP_DPP(m, m, 0x112, 0xf, false));
        m = max(m, TSP_DPP(m, m, 0x114, 0xf, false));
        m = max(m, TSP_DPP(m, m, 0x118, 0xf, false));
        m = max(m, TSP_DPP(m, m, 0x142, 0xa, false));
        m = max(m, TSP_DPP(m, m, 0x143, 0xc, false));
        carry = __builtin_amdgcn_readlane(m, 63);
        if constexpr (G == 16) m = __builtin_amdgcn_ds_bpermute(mine * 4, m);
        const int source = (m - 1) * 4;
        const int skip = (j0 + mine - __builtin_amdgcn_ds_bpermute(source, first)) * G;
        const int begin = __builtin_amdgcn_ds_bpermute(source, p) + skip;
        const int left = __builtin_amdgcn_ds_bpermute(source, len) - skip;
        const uint32_t bits = (uint32_t)__builtin_amdgcn_ds_bpermute(source, (int)own);
        const bool live = j0 + mine < total;
        const int byte = live ? (int)((uint32_t)begin * (uint32_t)sizeof(X)) : 0;
        const int about = live ? (int)((uint32_t)min(left, G) << 16 | bits) : 0;
        const int pieces = min(total - j0, 64);
        if constexpr (G == 16) {
            read_pieces(byte, about, pieces, from, use);
        } else {
            static_assert(G == 64, "a piece is a row of lanes or a wave");
            auto batch = [&](auto size, int t) {
                constexpr int kBatch = decltype(size)::value;
                uint32_t d[kBatch];
                X x[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    d[u] = (uint32_t)__builtin_amdgcn_readlane(about, t + u);
                    x[u] = *reinterpret_cast<const X *>(reinterpret_cast<const char *>(from) +
                                                        ((uint32_t)__builtin_amdgcn_readlane(byte, t + u) + (uint32_t)lane * (uint32_t)sizeof(X)));
                }
                use(x, d, (uint32_t)lane);
            };
            int t = 0;
            for (; t + 8 <= pieces; t += 8) batch(std::integral_constant<int, 8>{}, t);
            if (pieces - t >= 4) {
                batch(std::integral_constant<int, 4>{}, t);
                t += 4;
            }
            for (; t < pieces; ++t) batch(std::integral_constant<int, 1>{}, t);
        }
        wave_sync();
    }
}

// The segments of B behind up to kThreads entries of A, one per thread, cut into pieces of 16 elements that the waves share out
// evenly.
template <int kThreads>
struct SegmentList {
    static_assert((kThreads & (kThreads - 1)) == 0, "the search of stream_share stays inside the list");
    int first[kThreads];                                       // pieces before the segment
    uint2 at[kThreads];                                        // {first element, elements << 16 | 16 bits of its own}
};
// The segments of `entries` threads are in the list, `total` pieces; every wave streams its share.
template <int kThreads, typename X, typename Use>
__device__ __forceinline__ void stream_share(const SegmentList<kThreads> &list, int entries, int total, const X *from, Use &use) {
    constexpr int kWaves = kThreads / 64;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int half = entries > 1 ? 1 << (31 - __builtin_clz(entries - 1)) : 0;     // the largest power of two below them
    const int share = (total + 4 * kWaves - 1) / (4 * kWaves) * 4, end = min((wave + 1) * share, total);
    int at = 0;                                                // the last segment that begins at or before the lane's piece
    for (int j0 = wave * share; j0 < end; j0 += 64) {
        const int j = j0 + 4 * (lane % 16) + lane / 16;        // the piece this lane describes (read_pieces)
        // Few segments begin between the last piece described before and the next round's, and the search goes no further; where 64 do
        // it is of all of the list.  (Up to ten looks, one waiting for the other, without it: the sizing of the large rows of R-MAT scale
        // 18 3.49 -> 3.27 ms.)
        int most = half;
        if (j0 > wave * share) {
            at = __builtin_amdgcn_readlane(at, 63);
            const int k = at + 1 + lane;
            const int near = __popcll(__ballot((k < entries) & (list.first[min(k, kThreads - 1)] < j0 + 64)));
            if (near < 64) most = near ? 1 << (31 - __builtin_clz(near)) : 0;
            else at = 0;
        }
        for (int d = most; d > 0; d >>= 1)
            if ((at + d < kThreads) & (list.first[min(at + d, kThreads - 1)] <= j)) at += d;
        const uint2 x = list.at[at];
        const int skip = (j - list.first[at]) * 16;
        const bool live = j < end;
        read_pieces(live ? (int)((x.x + (uint32_t)skip) * (uint32_t)sizeof(X)) : 0,
                    live ? (int)((uint32_t)min((int)(x.y >> 16) - skip, 16) << 16 | (x.y & 0xFFFFu)) : 0, min(end - j0, 64), from, use);
    }
}

struct CountArgs {
    const int32_t *heavy;
    int64_t heavy_cap;
    const int64_t *d_scalars;
    const int32_t *a_start, *b_start;
    const int2 *a_rec;
    const uint32_t *b_word;
    const int32_t *b_words;
    const int32_t *b_spans;              // k_heavy_pack's span_table
    int32_t b_nnz;
    int windows;                         // of kWin columns each
    int spans;
    int span_windows;                    // windows whose bits the block's LDS holds
    int32_t *row_nnz;                    // null: only the pattern is wanted
    uint32_t *group_len;
    uint32_t *offset;                    // [heavy][windows] entries of the row before each window
    int heavy_from;                      // the rows of this launch begin here
    uint32_t *bits;                      // [heavy - heavy_from][windows][kWin / 32]; or null
    // The launch for the large rows goes by the first of the tasks that each has in the list of k_heavy_fill, the other one by
    // `heavy`; that leaves out rows of so many products (0: none).
    const int4 *tasks;
    int64_t n_large;
    const int32_t *ub;
    int large_products;
};

// A block per heavy row ORs the words of the rows of B behind it into one bit per column in LDS; OR is free of order, so
// the row may be spread over the block: by pieces of 16 words where every thread has at most one entry of A, else entry i of
// the row of A goes to wave i mod the number of waves that get 16 and more.
// Large rows have blocks of 1024 threads, the others, which are bound by the block's own steps, of 256, or of 512 where C is so
// wide that the LDS holds four blocks (scale 18 1.54 -> 1.39 ms; scale 16, whose bits are an eighth, 135 -> 220 us).  All rows
// by 256 threads: R-MAT scale 14 88 us, split 33 + 28; scale 18 5.3 ms, split 3.4 + 1.4.  All by the threads of the light ones,
// the products of scale 13 / 14 / 16 / 18: 158 / 294 / 2397 / 19,360 us, split 155 / 273 / 2235 / 19,720.  No more than 80 scalar
// registers: with the 106 that the compiler takes otherwise a SIMD has 7 waves, and a CU one block of 1024 threads (4.6 instead
// of 3.9 ms).
// Bound by round trips to the words: with all words from 2 MB 2.75 instead of 3.7 ms, without the LDS additions no less, with
// words of half the bytes, or twice as many in flight, no less either.
template <int kWin, int kThreads, bool kLargeRows>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_heavy_count(const CountArgs a) {
    extern __shared__ __align__(16) uint32_t bits[];
    constexpr int kWaves = kThreads / 64;
    __shared__ union {
        uint32_t mark[kWaves][64];
        SegmentList<kThreads> segment;
    } s_list;
    __shared__ int s_total[kWaves];
    __shared__ uint32_t s_cnt[kSpanWindows];
    __shared__ uint32_t s_run;
    constexpr int kWords = kWin / 32, kPerLane = kWords / 64;
    int64_t h;
    int32_t row;
    // (the lists of a product whose numbers the host does not have yet may be shorter than the launch)
    if constexpr (kLargeRows) {
        const int64_t t = min(a.n_large, uniform_load(a.d_scalars + S_ROW_LARGE_TASKS)) - 1 - (int64_t)blockIdx.x;
        if (t < 0) return;
        const int4 task = a.tasks[t];
        if (task.z != 0) return;
        row = __builtin_amdgcn_readfirstlane(task.x);
        h = __builtin_amdgcn_readfirstlane(task.y);
        if (h >= a.heavy_cap) return;
    } else {
        h = a.heavy_from + (int64_t)blockIdx.x;
        if (h >= a.heavy_cap || (a.d_scalars && h >= uniform_load(a.d_scalars + S_ROW_LISTS) >> 36)) return;
        row = uniform_load(a.heavy + h);
        if (a.large_products > 0 && uniform_load(a.ub + row) >= a.large_products) return;
    }
    const int32_t s = uniform_load(a.a_start + row), e = uniform_load(a.a_start + row + 1);
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int w = threadIdx.x; w < a.span_windows * kWords + 64; w += kThreads) bits[w] = 0;
    if (threadIdx.x == 0) s_run = 0;
    const bool even = e - s <= kThreads;
    const int dealt = min(kWaves, (e - s + 15) / 16);
    for (int w0 = 0; w0 < a.windows; w0 += a.span_windows) {
        const int w1 = min(w0 + a.span_windows, a.windows);
        const uint32_t words = (uint32_t)(w1 - w0) * kWords;
        auto segment = [&](int32_t k, int32_t *len) {        // of entry k of A
            const int32_t c = a.a_rec[k].x;
            if (a.b_spans) {
                const int32_t *ends = a.b_spans + ((int64_t)c * (a.spans + 1) + w0 / kSpanWindows);
                const int32_t p = max(ends[0], 0);           // (in bounds whatever an operand that was not validated holds)
                *len = min(ends[1], a.b_nnz) - p;
                return p;
            }
            *len = a.b_words[c];
            return a.b_start[c];
        };
        const uint32_t nothing = ((uint32_t)a.span_windows * kWords + lane) * 4;       // (for lanes without an element)
        auto use = [&](const auto &x, const auto &d, uint32_t l) {
            // (inside the bits whatever the operand holds: k_row_prepare leaves no column beyond B's, and a block has room for
            // all kSpanWindows windows where there are more of them)
#pragma unroll
            for (size_t u = 0; u < sizeof(x) / sizeof(x[0]); ++u) {
                const uint32_t byte = (x[u] & (uint32_t)(kSpanWindows * kWords * 2 - 2)) << 1, half = x[u] << 4;
                const uint32_t columns = (x[u] >> 16) << (half & 31u);
                atomicOr(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(bits) + (l < d[u] >> 16 ? byte : nothing)), columns);
            }
        };
        if (even) {
            // (of a row of B of more than 65,535 words the rest is a segment for the same thread's next turn)
            int32_t p = 0, len = 0;
            const int32_t k = s + (int32_t)threadIdx.x;
            if (k < e) p = segment(k, &len);
            do {
                const int32_t now = min(max(len, 0), 0xFFFF);
                const int pieces = (now + 15) / 16, inc = (int)wave_inclusive_scan((uint32_t)pieces);
                if (lane == 63) s_total[wave] = inc;
                __syncthreads();
                const int to = row16_inclusive_scan(lane % 16 < kWaves ? s_total[lane % 16] : 0);
                s_list.segment.first[threadIdx.x] = inc - pieces + (wave > 0 ? __builtin_amdgcn_readlane(to, wave - 1) : 0);
                s_list.segment.at[threadIdx.x] = make_uint2((uint32_t)p, (uint32_t)now << 16);
                __syncthreads();
                stream_share<kThreads>(s_list.segment, e - s, __builtin_amdgcn_readlane(to, kWaves - 1), a.b_word, use);
                p += now;
                len -= now;
            } while (__syncthreads_or(len > 0));
        } else {
            __syncthreads();
            for (int32_t base = s; base < e && wave < dealt; base += 64 * dealt) {
                const int32_t k = base + lane * dealt + wave;
                int32_t p = 0, len = 0;
                if (k < e) p = segment(k, &len);
                stream_pieces<16, uint32_t>(p, len, 0u, a.b_word, s_list.mark[wave], use);
            }
        }
        __syncthreads();
        for (int w = wave; w < w1 - w0; w += kWaves) {
            uint32_t n = 0, word[kPerLane];
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
                uint32_t *at = &bits[w * kWords + i * 64 + lane];
                word[i] = *at;
                n += __popc(word[i]);
                *at = 0;
            }
            n = wave_sum(n);
            if (a.bits)
#pragma unroll
                for (int i = 0; i < kPerLane; ++i)
                    a.bits[((h - a.heavy_from) * a.windows + w0 + w) * kWords + i * 64 + lane] = word[i];
            if (lane == 0) s_cnt[w] = n;
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t n = lane < w1 - w0 ? s_cnt[lane] : 0;
            const uint32_t inc = wave_inclusive_scan(n), before = s_run;
            if (lane < w1 - w0 && a.row_nnz) a.offset[h * a.windows + w0 + lane] = before + inc - n;
            if (lane == 63) s_run = before + inc;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && a.row_nnz) {
        a.row_nnz[row] = (int32_t)s_run;
        atomicAdd(&a.group_len[row / T], s_run);
    }
}

struct FillArgs {
    const int4 *tasks;                   // [task_cap]: the large ones, then others or nothing, then the light ones
    int64_t n_tasks, n_large, task_cap;
    bool large, light;                   // which of them this launch is for
    const int32_t *a_start, *b_start;
    const int2 *a_rec;
    const uint32_t *pack;
    const int32_t *table;
    int32_t b_nnz;
    int windows;
    const uint32_t *offset;
    const uint32_t *bits;                // pattern of heavy rows [heavy_from, heavy_to) of C from the sizing pass
    int heavy_from, heavy_to;
    const int64_t *c_row_ptr;
    int32_t *c_col;
    float *c_val;
    int window_shift;
    float p_scale, c_scale;              // integers from the products, values from the integer sums
    const int32_t *live;                 // of k_row_finish, or null
};

// A block per task: a row of C, or some of its windows, a step at a time: as many windows as hold at most kCap entries
// and kSpanColumns columns.  The pattern of the step, a bit per column, is known from the sizing pass, so its entries
// have places of their own in LDS: column c's is the number of bits before it, looked up as {32 bits, entries before
// them}.  The waves stream the segments of B behind the row and add the products at their places; then the values go out
// as they lie, and the columns, listed from the bits.  (A dense accumulator per window of 8192 columns needs no look-up but
// up to 32 steps for a row, most of them nearly empty.)
// Where every thread has at most one entry of A, a step's segments are cut into pieces of 16 elements and every wave takes as
// many of them as the others, whichever segments they belong to.  (Dealt by entries of A, 64 apiece, the busiest wave had
// 1.9 times the mean on R-MAT scale 18, 2.9 times on rows of 37 entries, and the others waited for it.)  Longer rows are
// dealt by entries: many of them meet each wave.  What the next step needs of the pattern and of the segments' ends is
// requested before this one's entries go out.
// 64 registers and nothing in scratch memory, so that 8 waves per SIMD hide the round trips to the elements of B: R-MAT
// scale 18 18.9 -> 16.4 ms (20 to 90 bytes of scratch: 17.2 to 26), 4100 rows of 37 entries 52 -> 44 us.  The vector
// ALUs are busy 63 %, half of it not with products but with what a step costs by its windows; LDS 37 %.  Traffic past the
// L2 caches (82 GB read, 24 GB written) does not bind it: with all elements of B from 2 MB 5 % less.  Entries go out four to a
// thread (16.5 -> 16.3 ms).
//
// The accumulator: LDS adds an fp32 number one lane after the other (193 cycles for a wave's 64 lanes, measured), an
// integer or an fp64 number all lanes at a time (5, 8 and 8 to 16 cycles for 32-bit and 64-bit integers and fp64).  So
// the sums are integers where they are exact in them, and fp64 otherwise; fp64 only with a block of one wave, whose
// steps follow one another (lanes of a step that meet at an entry are added by the LDS one after the other).  64-bit
// integers: p * 2^k + 1.5 * 2^52 in fp64 holds the integer p * 2^k in its low bits (|p * 2^k| < 2^51).
constexpr int kSpanColumns = 1 << 16;    // the elements of B hold 16 bits of the column
// The table of a C of at most so many columns is a quarter as long, which is what many light rows spend their time on:
// 6000 rows of 60 entries, 6000 columns, 139 -> 119 us; with more columns a row takes more steps (R-MAT scale 17, 2.75 ->
// 3.05 ms with a table of 32768 columns, 3.67 with one of 16384; scales 13 and 14 the same with either).
constexpr int kNarrowColumns = 1 << 14;
// Rows of so many products, summed in 32 bits, are large: blocks of 1024 threads and steps of 12,288 entries, two blocks to a
// CU.  A step costs every wave some 330 vector instructions whatever it holds, so that rows of many entries want few steps, and
// rows of few entries few waves.  R-MAT scale 18, all rows by 512 threads and 4096 entries 16.3 ms, all by 1024 15.2, large from
// 8192 / 16,384 / 32,768 products on 14.75 / 14.5 / 14.1; scale 14 (a table for few columns) 235 us, 230, 184 / 178 / 188, and
// 168 with blocks of 256 threads for the light ones.
constexpr int kLarge = 32768, kLargeNarrow = 16384;
// ... in products of so many intermediate ones at least: two launches more pay where they fill the chip.  The products of R-MAT
// graphs without them and with them, us: of scale 10 and 11 (1.9 and 3.3 million intermediate products) 64 / 83 and 68 / 83,
// 12 (6.9 and 9.5 million) 87 / 100 and 89 / 104, 13 (27 million) 148 / 155, 14 (101 million) 308 / 273, 16 (1.2 billion)
// 2452 / 2235, 18 21,860 / 19,720.  (The line was set when more than one kernel was slower; the two meet between 27 and 101 million
// now.)
constexpr int64_t kSplitProducts = 8 << 20;

template <typename Acc, int kCap, int kThreads, int kSpan, int kPiece = 16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kThreads == 64 ? 1 : 8, 8))) void k_heavy_fill(const FillArgs a) {
    constexpr int kWaves = kThreads / 64, kWords = kSpan / 32;
    // (before the entries a place for a column that the pattern does not have; 16 bytes, and behind them as many that are written too)
    constexpr int kPad = 16 / (int)sizeof(Acc);
    __shared__ __align__(16) Acc padded[kPad + kCap + kPad];
    Acc *const acc = padded + kPad;
    __shared__ __align__(16) int2 places[kWords];              // {bits of 32 columns, entries before them, less one}
    __shared__ union {
        uint32_t mark[kWaves][64];                             // of stream_pieces
        SegmentList<kThreads> segment;                         // (with the value of A)
    } s_list;
    __shared__ int2 s_total[kWaves];                           // of a wave's threads: {entries of C, pieces}
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    auto sync = [] {
        if constexpr (kThreads == 64) wave_sync();
        else __syncthreads();
    };
    // (what is derived from the thread's number is made again in every part of a step: kept over the reading of B it would take
    // the registers that the elements in flight need)
    auto thread = [] {
        int t = (int)threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    if (a.live && !uniform_load(a.live)) return;
    const int64_t n_large = a.live ? uniform_load(a.live + 2) : a.n_large, n_light = (a.live ? uniform_load(a.live + 1) : a.n_tasks) - n_large;
    int64_t t = blockIdx.x;
    if (!a.large || t >= n_large) {
        t -= a.large ? n_large : 0;
        if (!a.light || t >= n_light) return;
        t += a.task_cap - n_light;
    } else {
        t = n_large - 1 - t;                                   // (see there)
    }
    const int32_t row = uniform_load(&a.tasks[t].x), heavy = uniform_load(&a.tasks[t].y);
    int w = uniform_load(&a.tasks[t].z);
    const int w_end = uniform_load(&a.tasks[t].w);
    const int32_t s = uniform_load(a.a_start + row), deg = uniform_load(a.a_start + row + 1) - s;
    const int64_t row_first = uniform_load(a.c_row_ptr + row);
    const uint32_t row_len = (uint32_t)(uniform_load(a.c_row_ptr + row + 1) - row_first);
    if (heavy < a.heavy_from || heavy >= a.heavy_to || deg <= 0 || w >= w_end) return;
    // No element finds a place outside acc, whatever an operand that was not validated holds: the words of a step have no more entries
    // than it has, and those that are not of a step yet have none.
    for (int i = threadIdx.x; i < kWords; i += kThreads) places[i] = make_int2(0, -1);
    sync();
    const uint32_t *offset = a.offset + (int64_t)heavy * a.windows;
    const int word_shift = a.window_shift - 5;                 // words per window
    const uint32_t *kept = a.bits + (((int64_t)(heavy - a.heavy_from) * a.windows) << word_shift);
    const bool one = a.table == nullptr;
    const bool even = kWaves > 1 && deg <= kThreads;
    const int dealt = min(kWaves, (deg + 15) / 16);            // waves that take entries of A, where they are dealt
    // (in bounds whatever an operand that was not validated holds)
    const int32_t *ends_of = one ? a.b_start : a.table;        // where the segments of a row of B begin and end, from ends_at() on
    auto ends_at = [&](int32_t column) { return one ? (uint32_t)column : (uint32_t)column * (uint32_t)(a.windows + 1); };
    auto begin_in = [&](uint32_t at, int v) { return max(element(ends_of, at + (uint32_t)(one ? 0 : v)), 0); };
    auto end_in = [&](uint32_t at, int v_end) { return min(element(ends_of, at + (uint32_t)(one ? 1 : v_end)), a.b_nnz); };
    auto value_bits = [](const int2 &x) -> uint32_t { return __builtin_bit_cast(uint16_t, (_Float16)__uint_as_float((uint32_t)x.y)); };
    // lane i: entries of the row up to the end of window ends_from + i
    int ends_from = w;
    auto window_ends = [&] { return ends_from + lane + 1 < a.windows ? offset[ends_from + lane + 1] : row_len; };
    uint32_t ends = window_ends(), first = uniform_load(offset + w), next_first;
    int w_next;
    // the windows of the step that begins at w: as many as hold at most kCap entries and kSpan columns
    auto end_of_step = [&] {
        if (w - ends_from + (kSpan >> a.window_shift) > 64) {
            ends_from = w;
            ends = window_ends();
        }
        const int at_window = ends_from + lane;
        const bool fits = at_window >= w && at_window < w_end && at_window - w < (kSpan >> a.window_shift) && ends - first <= (uint32_t)kCap;
        w_next = w + max(__popcll(__ballot(fits)), 1);
        next_first = (uint32_t)__builtin_amdgcn_readlane((int)ends, w_next - 1 - ends_from);
    };
    // This thread's entry of A, where each has one: its value, and where its segment of B in the step begins and ends
    const bool mine = even && (int)threadIdx.x < deg;
    uint32_t my_value = 0, my_ends = 0;
    int my_begin = 0, my_end = 0;
    if (mine) {
        const int2 x = a.a_rec[s + (int)threadIdx.x];
        my_ends = ends_at(x.x);
        my_value = value_bits(x);
        my_begin = begin_in(my_ends, w);
    }
    end_of_step();
    uint4 b = make_uint4(0, 0, 0, 0);                          // four words of the step's pattern (of its first, with one wave)
    auto request = [&] {
        if (mine) my_end = end_in(my_ends, w_next);
        const int at = thread() * 4;
        b = make_uint4(0, 0, 0, 0);
        if (at < (w_next - w) << word_shift) b = *reinterpret_cast<const uint4 *>(kept + ((int64_t)w << word_shift) + at);
    };
    request();
    while (w < w_end) {
        const int some = (int)min(next_first - first, (uint32_t)kCap);
        const int w0 = w, w1 = w_next, p = my_begin;
        const uint32_t from = first;
        auto next_step = [&] {                                 // its requests are on their way while this step's entries go out
            my_begin = max(my_end, 0);
            w = w_next;
            first = next_first;
            if (w < w_end) {
                end_of_step();
                request();
            }
        };
        if (some > 0) {
            int pieces = 0;
            uint32_t about = 0;
            if (mine) {
                const int len = min(max(my_end - p, 0), 0xFFFF);
                about = (uint32_t)len << 16 | my_value;
                pieces = (len + kPiece - 1) / kPiece;
            }
            // places of the step's entries, four words per thread and round, and of its pieces
            const int words = (w1 - w0) << word_shift;
            int run = 0, total_pieces = 0;
            static_assert(kWaves == 1 || kWords <= kThreads * 4, "one round");
            const int tid = thread();
            for (int i = tid; i * 16 < some * (int)sizeof(Acc); i += kThreads)
                reinterpret_cast<int4 *>(acc)[i] = make_int4(0, 0, 0, 0);
            for (int base = 0; base < words; base += kThreads * 4) {
                const int at = base + tid * 4;
                if (base > 0) {
                    b = make_uint4(0, 0, 0, 0);
                    if (at < words) b = *reinterpret_cast<const uint4 *>(kept + ((int64_t)w0 << word_shift) + at);
                }
                const int n0 = __popc(b.x), n1 = n0 + __popc(b.y), n2 = n1 + __popc(b.z), n3 = n2 + __popc(b.w);
                const int inc = (int)wave_inclusive_scan((uint32_t)n3);
                int before = run + inc - n3 - 1;
                if constexpr (kWaves > 1) {
                    const int pieces_inc = (int)wave_inclusive_scan((uint32_t)pieces);
                    int pieces_before = pieces_inc - pieces;
                    if (lane == 63) s_total[wave] = make_int2(inc, pieces_inc);
                    __syncthreads();
                    // (sums over the waves, which are fewer than a row of lanes)
                    const int2 total = tid % 16 < kWaves ? s_total[tid % 16] : make_int2(0, 0);
                    const int entries_to = row16_inclusive_scan(total.x), pieces_to = row16_inclusive_scan(total.y);
                    if (wave > 0) {
                        before += __builtin_amdgcn_readlane(entries_to, wave - 1);
                        pieces_before += __builtin_amdgcn_readlane(pieces_to, wave - 1);
                    }
                    total_pieces = __builtin_amdgcn_readlane(pieces_to, kWaves - 1);
                    if (even) {
                        s_list.segment.first[tid] = pieces_before;
                        s_list.segment.at[tid] = make_uint2((uint32_t)p, about);
                    }
                } else {
                    run += __builtin_amdgcn_readlane(inc, 63);
                }
                if (at < words) {
                    int4 *to = reinterpret_cast<int4 *>(places + (((w0 << word_shift) + at) & (kWords - 1)));
                    to[0] = make_int4((int)b.x, before, (int)b.y, before + n0);
                    to[1] = make_int4((int)b.z, before + n1, (int)b.w, before + n2);
                }
            }
            sync();
            const uint32_t c0 = (uint32_t)w0 << a.window_shift;
            // (all look-ups of a batch before the first addition, and nothing selected but whether a lane adds: a chain of
            // look-up and addition for every element leaves the LDS idle for the latency of both)
            auto use = [&](const auto &x, const auto &d, uint32_t l) {
                constexpr int kBatch = (int)(sizeof(x) / sizeof(x[0]));
                int2 place[kBatch];
                int at[kBatch];
                float product[kBatch];
                // (the compiler would move a load to the only lanes that use it, behind the branch below, and wait there for its round trip:
                // light rows of R-MAT scale 18 4.14 -> 3.89 ms, 4099 rows of 37 entries 44.2 -> 41.6 us)
                auto keep = [](auto &v) { asm volatile("" : "+v"(v)); };
                uint32_t element[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    element[u] = x[u];
                    keep(element[u]);
                    place[u] = *reinterpret_cast<const int2 *>(reinterpret_cast<const char *>(places) + ((element[u] >> 2) & (uint32_t)(kWords - 1) * 8u));
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    keep(place[u].x);
                    keep(place[u].y);
                    // (inside acc also for a column that the pattern does not have: at most one before it, `places` says)
                    at[u] = __popc((uint32_t)place[u].x << (element[u] & 31u)) + place[u].y;
                    // the product of two fp16 numbers is exact; + 0 makes a positive zero of a negative one
                    product[u] = __builtin_fmaf((float)__builtin_bit_cast(_Float16, (uint16_t)(element[u] >> 16)),
                                                (float)__builtin_bit_cast(_Float16, (uint16_t)d[u]), 0.f);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const bool active = l < d[u] >> 16;
                    if constexpr (std::is_floating_point<Acc>::value) {
                        if (active) unsafeAtomicAdd(&acc[at[u]], (double)product[u]);
                    } else if constexpr (sizeof(Acc) == 4) {
                        const int whole = (int)(product[u] * a.p_scale);
                        if (active) atomicAdd(&acc[at[u]], whole);
                    } else {
                        const double shifted = __builtin_fma((double)product[u], (double)a.p_scale, 6755399441055744.0);
                        if (active)
                            atomicAdd(reinterpret_cast<unsigned long long *>(&acc[at[u]]),
                                      __builtin_bit_cast(unsigned long long, shifted) - 0x4338000000000000ull);
                    }
                }
            };
            if (even) {
                if constexpr (kWaves > 1) stream_share<kThreads>(s_list.segment, deg, total_pieces, a.pack, use);
            } else {
                for (int base = 0; base < deg && wave < dealt; base += 64 * dealt) {
                    const int k = base + (thread() & 63) * dealt + wave;
                    int begin = 0, len = 0;
                    uint32_t own = 0;
                    if (k < deg) {
                        const int2 x = a.a_rec[s + k];
                        const uint32_t at = ends_at(x.x);
                        begin = begin_in(at, w0);
                        len = end_in(at, w1) - begin;
                        own = value_bits(x);
                    }
                    stream_pieces<kPiece, uint32_t>(begin, len, own, a.pack, s_list.mark[wave], use);
                }
            }
            next_step();
            sync();
            float *to_val = a.c_val + row_first + from;
            struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };
            struct __attribute__((packed, aligned(4))) I4 { int x, y, z, w; };
            auto value = [&](Acc v) { return std::is_floating_point<Acc>::value ? (float)v : (float)v * a.c_scale; };
            struct alignas(16) A4 { Acc x, y, z, w; };
            const int t4 = thread() * 4, rest = some & ~3;
            for (int i = t4; i + 4 <= some; i += kThreads * 4) {
                const A4 v = *reinterpret_cast<const A4 *>(acc + i);
                *reinterpret_cast<F4 *>(to_val + (unsigned)i) = F4{value(v.x), value(v.y), value(v.z), value(v.w)};
            }
            if (t4 < (some & 3) * 4) to_val[(unsigned)(rest + t4 / 4)] = value(acc[rest + t4 / 4]);
            sync();
            int32_t *col = reinterpret_cast<int32_t *>(acc);
            for (int i = thread(); i < words; i += kThreads) {
                const int2 place = places[((w0 << word_shift) + i) & (kWords - 1)];
                uint32_t word = (uint32_t)place.x;
                int32_t *to = col + place.y;
                while (word) {
                    *++to = (int32_t)c0 + i * 32 + __ffs((int)word) - 1;
                    word &= word - 1;
                }
            }
            sync();
            int32_t *to_col = a.c_col + row_first + from;
            const int u4 = thread() * 4;
            for (int i = u4; i + 4 <= some; i += kThreads * 4) {
                const int4 c = *reinterpret_cast<const int4 *>(col + i);
                *reinterpret_cast<I4 *>(to_col + (unsigned)i) = I4{c.x, c.y, c.z, c.w};
            }
            if (u4 < (some & 3) * 4) to_col[(unsigned)(rest + u4 / 4)] = col[rest + u4 / 4];
            sync();
        } else {
            next_step();
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
    Tp *get_if_there(size_t n) {
        Tp *p = ctx_alloc_n<Tp>(ctx, n, s);
        if (p) blocks.push_back(p);
        return p;
    }
    template <typename Tp>
    Tp *get(size_t n) {
        Tp *p = get_if_there<Tp>(n);
        failed = failed || !p;
        return p;
    }
    void keep(void *p) { blocks.erase(std::find(blocks.begin(), blocks.end(), p)); }
    ~Workspace() {
        for (void *p : blocks) ctx_free(ctx, p, s);
    }
};

constexpr int kSampleRows = 128;         // tile-rows of an operand that are looked at
constexpr int kSampleEntries = 4096;     // ... and entries of each, at most
// A look pays where the pass over the operands takes long, and where a product by tiles is not out of the question: the pass
// takes 26 ns per thousand entries, the look and the launches that then find nothing to do 20 us together.
bool sample_pays(int64_t rows, int64_t nnz) { return nnz >= (1 << 18) && nnz > 8 * rows; }

// A wave per tile-row of up to two trips; longer ones get a block, four entries per thread in flight (the hub rows of a graph:
// one wave took 1.9 ms for the longest tile-row of an R-MAT graph of scale 18)
template <typename RP, typename VT>
bool wave_per_tile_row(const PrepareArgs<RP, VT> &a) {
    return a.nnz <= 128 * ((a.rows + T - 1) / T) && (size_t)a.bitmap_words * 16 <= 60 * 1024;
}
template <typename RP, typename VT>
void launch_prepare(const PrepareArgs<RP, VT> &a, bool long_rows, hipStream_t s) {
    const int64_t tile_rows = (a.rows + T - 1) / T;
    if (tile_rows == 0) return;
    if (wave_per_tile_row(a))
        hipLaunchKernelGGL((k_row_prepare<64, 2, RP, VT>), dim3((unsigned)((tile_rows + 3) / 4)), dim3(256),
                           (size_t)a.bitmap_words * 16, s, a, NoSecond{});
    else {
        auto launch = [&](auto kernel, int threads) { hipLaunchKernelGGL(kernel, dim3((unsigned)tile_rows), dim3(threads), (size_t)a.bitmap_words * 4, s, a, NoSecond{}); };
        // The longest tile-row, 3 ns per entry with 256 threads, keeps the launch waiting, where the last product of these sizes
        // had long rows: R-MAT scales 14 / 16 / 18 by 256 threads 64 / 197 / 515 us, by 512 43 / 120 / 345, by 1024 28 / 96 / 437.
        // (By 1024 with one, two and four entries of a thread in flight: scale 13 14.8 / 16.3 / 15.3, 14 27.4 / 30.1 / 28.5, 15 38.8 /
        // 41.5 / 43.4, 16 81 / 84 / 94: it is the instructions of one CU that bind.)
        // (Even rows, 80,000 of 12 entries: 20, 30, 38.)
        if (!long_rows) launch(k_row_prepare<256, 4, RP, VT>, 256);
        else if (tile_rows <= 4096) launch(k_row_prepare<1024, 1, RP, VT>, 1024);
        else launch(k_row_prepare<512, 4, RP, VT>, 512);
    }
}
// Two operands go in one launch of k_row_prepare, whose blocks all have the wider one's bitmaps, where neither has less than three
// quarters of the blocks on a CU for that which it has on its own (registers are for eight; bitmaps of a block in bytes).  A of
// 262,144 rows and 4000 columns times B of 4000 rows and 700,000 / 800,000 / 1,000,000 / 1,900,000 columns (7, 6, 5, 2 blocks):
// apart 21 us each, at once 18 / 18 / 22 / 34; 20,000 rows times B of 700,000 / 800,000 / 1,000,000 / 1,900,000 rows and 1000
// columns: apart 31 / 33 / 38 / 61, at once 27 / 32 / 49 / 151; by 256 threads a tile-row, 3, 4 and 7.8 million columns (6, 5, 2):
// apart 22, at once 21 / 23 / 42.
constexpr int prepare_blocks_per_cu(size_t bitmaps) { return (int)std::min<size_t>(8, 160 * 1024 / (bitmaps + 1024)); }
constexpr bool prepare_at_once(size_t a_bitmaps, size_t b_bitmaps) {
    return 4 * prepare_blocks_per_cu(std::max(a_bitmaps, b_bitmaps)) >= 3 * prepare_blocks_per_cu(std::min(a_bitmaps, b_bitmaps));
}
static_assert(prepare_at_once(64, 64) && prepare_at_once(64, 25 * 1024) && !prepare_at_once(64, 26 * 1024) && !prepare_at_once(64, 60 * 1024));
static_assert(!prepare_at_once(60 * 1024, 64) && prepare_at_once(59 * 1024, 60 * 1024), "whichever is the wide one");
template <typename RP, typename VT>
void launch_prepare_both(const PrepareArgs<RP, VT> &a, const PrepareArgs<RP, VT> &b, bool long_rows, hipStream_t s) {
    const int64_t a_tile_rows = (a.rows + T - 1) / T, b_tile_rows = (b.rows + T - 1) / T;
    const bool waves = wave_per_tile_row(a);
    const int teams = prepare_teams(waves ? 64 : 256);
    if (a_tile_rows == 0 || b_tile_rows == 0 || waves != wave_per_tile_row(b) || (!waves && long_rows) ||
        !prepare_at_once((size_t)a.bitmap_words * 4 * teams, (size_t)b.bitmap_words * 4 * teams)) {
        launch_prepare(a, long_rows, s);
        launch_prepare(b, false, s);
        return;
    }
    const uint32_t a_blocks = (uint32_t)((a_tile_rows + teams - 1) / teams), b_blocks = (uint32_t)((b_tile_rows + teams - 1) / teams);
    hipLaunchKernelGGL((waves ? k_row_prepare<64, 2, RP, VT, Second<RP, VT>> : k_row_prepare<256, 4, RP, VT, Second<RP, VT>>), dim3(a_blocks + b_blocks), dim3(256),
                       (size_t)std::max(a.bitmap_words, b.bitmap_words) * 4 * teams, s, a, Second<RP, VT>{b, a_blocks});
}

// What k_row_prepare needs beyond the operand, for A (null members for B)
struct LeftOperand {
    int32_t *ub;
    uint32_t *rows_of, *part_len;
    unsigned long long *products;
    const tsp_csr *B;
    SmallShape shape;
    int windows;
    int32_t *heavy;
    int4 *tasks;
    int large_products;
    bool long_rows;                      // by the last product of these sizes
    int64_t heavy_cap, task_cap;
};

// A, and B unless it is null or A itself
void prepare(tsp_context *ctx, const tsp_csr *A, const RowMatrix &a_out, const LeftOperand &left, const tsp_csr *B, const RowMatrix &b_out,
             hipStream_t s, const int64_t *skip) {
    auto args = [&](auto rp, auto v, const tsp_csr *M, const RowMatrix &out) {
        using RP = decltype(rp);
        using VT = decltype(v);
        PrepareArgs<RP, VT> a{};
        a.row_ptr = static_cast<const RP *>(M->row_ptr);
        a.col = M->col_idx;
        a.val = static_cast<const VT *>(M->val);
        a.rows = M->rows;
        a.cols = M->cols;
        a.nnz = M->nnz;
        a.bitmap_words = (int)((M->cols + T * 32 - 1) / (T * 32) + 3) & ~3;
        a.validate = ctx->validate;
        a.out = out;
        if (M == A) {
            a.ub = left.ub;
            a.products = left.products;
            a.b_row_ptr = left.B->row_ptr;
            a.b_is_i64 = left.B->row_ptr_type == TSP_I64;
            a.b_rows = left.B->rows;
            a.b_nnz = (int32_t)left.B->nnz;
            a.small_lanes = left.shape.lanes;
            a.small_products = left.shape.products;
            a.windows = left.windows;
            a.heavy = left.heavy;
            a.tasks = left.tasks;
            a.large_products = left.large_products;
            a.heavy_cap = left.heavy_cap;
            a.task_cap = left.task_cap;
            a.rows_of = left.rows_of;
            a.part_len = left.part_len;
        }
        a.d_scalars = ctx->d_scalars;
        a.skip = skip;
        return a;
    };
    auto of_types = [](const tsp_csr *M, auto run) {
        const bool f16 = M->val_type == TSP_F16;
        if (M->row_ptr_type == TSP_I32) f16 ? run(int32_t{}, uint16_t{}) : run(int32_t{}, float{});
        else f16 ? run(int64_t{}, uint16_t{}) : run(int64_t{}, float{});
    };
    const bool both = B && B != A && A->row_ptr_type == B->row_ptr_type && A->val_type == B->val_type;
    of_types(A, [&](auto rp, auto v) {
        if (both) launch_prepare_both(args(rp, v, A, a_out), args(rp, v, B, b_out), left.long_rows, s);
        else launch_prepare(args(rp, v, A, a_out), left.long_rows, s);
    });
    if (B && B != A && !both) of_types(B, [&](auto rp, auto v) { launch_prepare(args(rp, v, B, b_out), false, s); });
}

void launch_fill(FillArgs &f, FillKind kind, bool short_rows, bool split, hipStream_t s) {
    auto launch = [&](auto kernel, int threads, bool large, bool light) {
        f.large = large;
        f.light = light;
        const int64_t blocks = (large ? f.n_large : 0) + (light ? f.n_tasks - f.n_large : 0);
        if (blocks > 0) hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, s, f);
    };
    f.p_scale = std::ldexp(1.0f, -kind.scale);
    f.c_scale = std::ldexp(1.0f, kind.scale);
    const bool narrow = (int64_t)f.windows << f.window_shift <= kNarrowColumns;
    if (kind.sum == FillKind::kInt32 && !split) {
        launch(narrow ? k_heavy_fill<int32_t, 4096, 512, kNarrowColumns> : k_heavy_fill<int32_t, 4096, 512, kSpanColumns>, 512, true, true);
    } else if (kind.sum == FillKind::kInt32 && narrow) {
        launch(k_heavy_fill<int32_t, 12288, 1024, kNarrowColumns>, 1024, true, false);
        launch(k_heavy_fill<int32_t, 4096, 256, kNarrowColumns>, 256, false, true);
    } else if (kind.sum == FillKind::kInt32) {
        launch(k_heavy_fill<int32_t, 12288, 1024, kSpanColumns>, 1024, true, false);
        launch(k_heavy_fill<int32_t, 4096, 512, kSpanColumns>, 512, false, true);
    } else if (kind.sum == FillKind::kInt64 && narrow) {     // (4100 rows of 37 entries: 44 us with 512 threads, 42 with 256)
        launch(k_heavy_fill<long long, 4096, 256, kNarrowColumns>, 256, true, true);
    } else if (kind.sum == FillKind::kInt64) {
        launch(k_heavy_fill<long long, 4096, 512, kSpanColumns>, 512, true, true);
    } else {
        // (rows of B shorter than a wave: four at a time.  20,000 rows of 3 entries, five of 6600, normal values: 2338 -> 1285 us)
        launch(short_rows ? k_heavy_fill<double, 4096, 64, kSpanColumns, 16> : k_heavy_fill<double, 4096, 64, kSpanColumns, 64>, 64, true, true);
    }
}

}  // namespace

__global__ void k_clear_lists(int64_t *d_scalars) {
    if (threadIdx.x == 0) d_scalars[S_ROW_LISTS] = d_scalars[S_ROW_LARGE_TASKS] = 0;
}
__global__ void k_clear_arrivals(unsigned long long *counters, uint32_t *tile_counts) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    counters[i * kArriveStride] = 0;
    for (int k = i; k < kTileCounts; k += kArriveCounters) tile_counts[k] = 0;
}
// all but the count of products, which has run before anything else of the call
__global__ void k_clear_rows(int64_t *d_scalars, int64_t products) {
    if (threadIdx.x < kScalars) d_scalars[threadIdx.x] = threadIdx.x == S_PRODUCTS ? products : 0;
}

// Whether the row kernels are faster for A*B than the tile kernels: what the two take beyond the 30 us that both do, from
// times of 90 products of meshes, stencils, blocks, random and power-law graphs (in ns).  Those times, and all figures here, are of
// kernels before the present ones: small rows went through a hash table, and repeated products by tiles took more launches.  Small rows
// take less now (reckoned and timed: 65,536 rows of 8 random entries 68 and 40 us, a 512^2 mesh 89 and 45), repeated products by tiles up to
// 15 % less; the line has not been drawn again.  Rows: 13 per heavy row, 1 per
// thousand products, 8 where the heavy rows are summed in fp64 (3 on even rows, 8 to 20 on graphs), and 1 per thousand
// products of the small rows and lane of such a row.  Tiles: 19 us (more launches) and 0.15 per candidate pair of tiles, which
// is what they cost at least.  So a stencil or dense blocks go by tiles from 1500 rows on (27 points on a 24^3 grid: 69 us, by
// rows 157), a mesh, graph or random matrix by rows (a 300^2 mesh: 42 us, by tiles 68; 4000 rows of 73 entries at random: 105,
// 742).  Of the 90 the choice loses more than 6 % on three, 23 % on one.  Values of a normal distribution, which integers do not
// hold: 3000 rows, a fifth full, by rows 2469 us, by tiles 865; R-MAT scale 13 with 110 entries per row 5060, 3560; scale 18
// with 30 per row 98 ms, 207.
static bool rows_preferred(int64_t products, int64_t small_products, int lanes, int64_t heavy, bool integers, int64_t candidates) {
    return 13 * heavy + products / 1000 + (integers ? 0 : 7 * ((products - small_products) / 1000)) + lanes * (small_products / 1000) <=
           19000 + candidates / 20 * 3;
}

// The same from some of the tile-rows, a block each: what their rows cost by rows, and their tiles.  The pairs of tiles are
// estimated as the tiles of A times the mean tile-row of B.  On a graph, whose long tile-rows are met most, that is too low,
// by less than the distance at which it is a product by rows; elsewhere the tile kernels' own count shows it (tsp_spgemm).
// Clearly for tiles: by rows at least twice as long.  The kernels of the look at all tile-rows, launched behind this one, then
// have nothing to do, and the host waits for the end of it once either way.  10 us; first products of 131072 and of 24000
// rows of blocks 348 -> 235 and 150 -> 122 us.
struct SampleArgs {
    const void *row_ptr[2];              // of A and B, as the caller gave them
    const int32_t *col[2];
    int64_t rows[2], cols[2], nnz[2];
    int is_i64[2];
    int blocks[2];                       // tile-rows looked at (0 of B: A and B are one matrix)
    int small_lanes, small_products;
    int64_t *d_scalars;
};
__global__ __launch_bounds__(256) void k_row_sample(const SampleArgs a) {
    extern __shared__ uint32_t lds_bitmap[];
    __shared__ int32_t s_ptr[T + 1];
    __shared__ unsigned long long s_ub[T];
    __shared__ unsigned s_tiles;
    const int of = (int)blockIdx.x >= a.blocks[0], tid = threadIdx.x;
    const int64_t at = (int64_t)blockIdx.x - of * a.blocks[0], tile_rows = (a.rows[of] + T - 1) / T;
    const int64_t I = (2 * at + 1) * tile_rows / (2 * a.blocks[of]);
    auto pointer = [&](int m, int64_t i) {
        const int64_t p = a.is_i64[m] ? static_cast<const int64_t *>(a.row_ptr[m])[i] : static_cast<const int32_t *>(a.row_ptr[m])[i];
        return (int32_t)min(max(p, (int64_t)0), a.nnz[m]);
    };
    const int words = (int)((a.cols[of] + T * 32 - 1) / (T * 32));
    for (int w = tid; w < words; w += 256) lds_bitmap[w] = 0;
    if (tid <= T) {
        int32_t p = pointer(of, min(I * T + tid, a.rows[of]));
        p = max(p, TSP_DPP(p, p, 0x111, 0xf, false));
        p = max(p, TSP_DPP(p, p, 0x112, 0xf, false));
        p = max(p, TSP_DPP(p, p, 0x114, 0xf, false));
        p = max(p, TSP_DPP(p, p, 0x118, 0xf, false));
        p = max(p, TSP_DPP(p, p, 0x142, 0xa, false));
        s_ptr[tid] = p;
        if (tid < T) s_ub[tid] = 0;
    }
    if (tid == 0) s_tiles = 0;
    __syncthreads();
    const int32_t e0 = s_ptr[0], entries = s_ptr[T] - e0, n = min(entries, kSampleEntries);
    unsigned tiles = 0;
    for (int k0 = tid; k0 < n; k0 += 4 * 256) {
        int32_t c[4], len[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = a.col[of][e0 + min(k0 + u * 256, n - 1)];
            c[u] = (uint32_t)c[u] < (uint64_t)a.cols[of] ? c[u] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) len[u] = of ? 0 : min(max(pointer(a.blocks[1] ? 1 : 0, c[u] + 1) - pointer(a.blocks[1] ? 1 : 0, c[u]), 0), (1 << 25) - 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (k0 + u * 256 >= n) break;
            const int32_t k = e0 + k0 + u * 256;
            const uint32_t bit = 1u << ((c[u] >> 4) & 31);
            tiles += !(atomicOr(&lds_bitmap[c[u] >> 9], bit) & bit);
            if (of) continue;
            int r = 0;
#pragma unroll
            for (int step = T / 2; step >= 1; step >>= 1)
                if (s_ptr[r + step] <= k) r += step;
            atomicAdd(&s_ub[r], (unsigned long long)(uint32_t)len[u]);
        }
    }
    tiles = wave_sum(tiles);
    if (lane_id() == 0) atomicAdd(&s_tiles, tiles);
    __syncthreads();
    if (tid >= T) return;
    // (as if the rest of a longer tile-row were like its first entries)
    const double more = n > 0 ? (double)entries / n : 1.0;
    const int32_t ub = (int32_t)min(s_ub[tid], (unsigned long long)INT32_MAX);
    const bool small = small_row(s_ptr[tid + 1] - s_ptr[tid], ub, a.small_lanes, a.small_products);
    double cost = ub == 0 ? 0.0 : small ? (a.small_lanes + 1.0) * ub : 13000.0 + ub;        // rows_preferred, in ps
    for (int d = 1; d < T; d <<= 1) cost += __shfl_xor(cost, d, T);
    if (tid > 0) return;
    auto *scalars = reinterpret_cast<unsigned long long *>(a.d_scalars);
    atomicAdd(scalars + S_SAMPLE_TILES, (unsigned long long)(s_tiles * more) << (32 * of));
    if (!of) atomicAdd(scalars + S_SAMPLE_COST, (unsigned long long)(cost * more));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (before this block counts as done)
    if (atomicAdd(scalars + S_ROW_ARRIVED, 1ull) != gridDim.x - 1) return;
    const unsigned long long both = __hip_atomic_load(scalars + S_SAMPLE_TILES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long all = __hip_atomic_load(scalars + S_SAMPLE_COST, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double scale = (double)((a.rows[0] + T - 1) / T) / a.blocks[0], tiles_a = (double)(both & 0xFFFFFFFFull);
    const double mean_b = a.blocks[1] ? (double)(both >> 32) / a.blocks[1] : tiles_a / a.blocks[0];
    const double candidates = tiles_a * scale * mean_b;
    a.d_scalars[S_ROW_SKIP] = all * scale > 2.0 * (19e6 + 150.0 * candidates) ? (int64_t)candidates + 1 : 0;
    a.d_scalars[S_ROW_ARRIVED] = 0;
}

// What a run of the row kernels has come to
enum RowsEnd { kRowsNotTaken, kRowsTaken, kRowsAgain };     // (again: with other lanes, or with the operands prepared)

// A product of sizes whose last product had small rows only, straight from the operands (k_row_given).  Up to kGivenBlocks blocks of
// rows, whose numbers every block of k_given_finish adds up (64 KB for the last of them), and bitmaps of no more LDS than leaves a CU its
// eight blocks.  More blocks are left to the other kernels without having been timed.
constexpr int64_t kGivenBlocks = 16384;
constexpr size_t kGivenBitmaps = 16 * 1024;
constexpr int64_t kGivenRows = kGivenBlocks * 32, kGivenColumns = (int64_t)kGivenBitmaps / 16 * 32 * T;     // at most, of A
static_assert(kGivenColumns <= (int64_t)kTileCounts * T, "a count for every tile column of A");
static_assert(arrive_groups(kGivenBlocks) + arrive_groups(kGivenRows / T / 4) + arrive_groups(kGivenColumns / T / 4) <= kArriveCounters, "of the rows, the tiles of A and of B");
template <typename RP, typename VT>
static int rowwise_given(tsp_context *ctx, const tsp_csr *A, const tsp_csr *B, bool alias, tsp_csr *C, hipStream_t s, RowHint &hint,
                         const SmallShape &shape, int cost_lanes, RowsEnd *end) {
    const int64_t a_ntr = (A->rows + T - 1) / T, b_ntr = (B->rows + T - 1) / T;
    const int64_t row_blocks = (A->rows * shape.lanes + 255) / 256;
    const bool one_chunk = A->rows <= kChunkRows;
    Workspace ws{ctx, s, {}};
    GivenArgs<RP, VT> a{};
    // Counts of A's tiles in every tile column, where there are few of them (of the last product), or lists of them.  An addition is 0.11 ns
    // of the launch, a list three round trips more before the pairs are known; a row is 0.14 to 0.45 ns.  us, lists and counts: 37^2 mesh
    // (1.1 thousand tiles) 22.9 and 17.9, 1024 rows of 8 random entries (8 thousand) 24.7 and 19.2, A*P on 18^3 25.5 and 22.4, on 64^3 41.5
    // and 39.5, 512^2 mesh (180 thousand) 46.6 and 44.9; 12,725 and 65,536 rows of 8 random entries (8 tiles to a row) 28.3 and 39.9, 40.8
    // and 66.7.
    const bool counts = hint.a_tiles <= std::max<int64_t>(A->rows, 24576);
    auto tiles_of = [&](const tsp_csr *M, int64_t ntr, bool left) {
        TileArgs<RP> t{static_cast<const RP *>(M->row_ptr), M->col_idx, M->rows, M->cols, M->nnz, (int)((M->cols + T * 32 - 1) / (T * 32) + 3) & ~3, nullptr, nullptr, nullptr, nullptr};
        t.ntiles = ws.get<int32_t>((size_t)ntr);
        if (left) {                          // (memory for the lists either way: which way a product goes does not say whether there is enough)
            int32_t *const first = ws.get<int32_t>((size_t)ntr), *const tile_col = ws.get<int32_t>((size_t)M->nnz);
            if (counts) {
                t.counts = ctx->d_tile_counts;
            } else {
                t.first = first;
                t.tile_col = tile_col;
            }
        }
        return t;
    };
    a.a = tiles_of(A, a_ntr, true);
    a.per_wave = one_chunk ? 1 : 4;
    const int per_block = 4 * a.per_wave;
    a.a_blocks = (uint32_t)((a_ntr + per_block - 1) / per_block);
    if (!alias) {
        a.b = tiles_of(B, b_ntr, false);
        a.b_blocks = (uint32_t)((b_ntr + per_block - 1) / per_block);
    }
    a.a_tile_rows = a_ntr;
    a.b_tile_rows = b_ntr;
    a.b_ntiles = alias ? a.a.ntiles : a.b.ntiles;
    a.row_blocks = (uint32_t)row_blocks;
    a.pair_blocks = !counts ? (uint32_t)std::min<int64_t>(kPlanBlocks, (a_ntr + 15) / 16)
                  : one_chunk && b_ntr <= kPairsByOne ? 0u : (uint32_t)std::min<int64_t>(kPlanBlocks, (b_ntr + 255) / 256);
    a.validate = ctx->validate;
    a.looks = ctx->give_up ? 0u : kArriveSpins;
    a.counters = ctx->d_arrivals;
    a.operands = {static_cast<const RP *>(A->row_ptr), static_cast<const RP *>(B->row_ptr), A->col_idx, B->col_idx, static_cast<const VT *>(A->val),
                  static_cast<const VT *>(B->val), (int32_t)A->nnz, (int32_t)B->nnz, (uint32_t)(A->cols - 1), (uint32_t)(B->cols - 1)};
    SmallArgs &m = a.small;
    m.shape = shape;
    m.wave_bytes = (int)shape.wave_bytes();
    m.rows = A->rows;
    m.finish = one_chunk;
    m.row_nnz = ws.get<int32_t>((size_t)A->rows);
    m.found = ws.get<int2>((size_t)(row_blocks * (256 / shape.lanes) * shape.products));
    m.wave_total = ws.get<int32_t>((size_t)row_blocks * 4);
    m.block_len = ws.get<uint32_t>((size_t)row_blocks + 3);               // (read four at a time)
    int64_t *row_ptr = ws.get<int64_t>((size_t)A->rows + 1);
    const int64_t room = hint.nnz + std::min<int64_t>(hint.nnz / 16, 1 << 20);
    int32_t *col = ws.get<int32_t>((size_t)room), *live = one_chunk ? ws.get<int32_t>(1) : nullptr;
    float *val = ws.get<float>((size_t)room);
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;
    a.publish = GivenPublishArgs{A->rows, room, row_ptr, ctx->d_scalars, ctx->h_scalars_dev, ++ctx->publish_tag, live, alias};

    // (where blocks have given up, others have counted themselves, tiles and pairs after those had taken what was there)
    if (!ctx->arrivals_clean) hipLaunchKernelGGL(k_clear_arrivals, dim3(kArriveCounters / 256), dim3(256), 0, s, ctx->d_arrivals, ctx->d_tile_counts);
    ctx->arrivals_clean = false;
    phase_begin(ctx, TSP_PHASE_SYMBOLIC, s);
    {
        KernelTimer kt(ctx, TSP_KERNEL_SYM_COUNT, s);
        const size_t lds = std::max(4 * shape.wave_bytes() + SmallShape::kReadPast, (size_t)std::max(a.a.bitmap_words, a.b.bitmap_words) * 16);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.a_blocks + a.b_blocks + a.row_blocks + a.pair_blocks + 1u), dim3(256), lds, s, a); };
        // (two kernels: with both ways in one the lists cost 2 % on 12,725 rows of 8 entries)
        auto launch_for = [&](auto with) {
            constexpr bool kCounts = decltype(with)::value;
            if (shape.lanes == 8) launch(shape.narrow() ? k_row_given<8, true, kCounts, RP, VT> : k_row_given<8, false, kCounts, RP, VT>);
            else launch(shape.narrow() ? k_row_given<16, true, kCounts, RP, VT> : k_row_given<16, false, kCounts, RP, VT>);
        };
        if (counts) launch_for(std::true_type{});
        else launch_for(std::false_type{});
    }
    phase_end(ctx, TSP_PHASE_SYMBOLIC, s);
    CopyArgs copy{shape, A->rows, row_blocks * 4, nullptr, nullptr, m.found, m.wave_total, row_ptr, col, val, live};
    auto move = [&] { hipLaunchKernelGGL(k_small_copy, dim3((unsigned)row_blocks), dim3(256), 0, s, copy); };
    phase_begin(ctx, TSP_PHASE_NUMERIC, s);
    {
        KernelTimer kt(ctx, TSP_KERNEL_NUMERIC, s);
        auto launch = [&](auto kernel, int rows) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((A->rows + rows - 1) / rows)), dim3(256), 0, s, copy, row_ptr, m.row_nnz, m.block_len, room);
        };
        // (about 2000 entries to a block: see k_small_finish)
        const int64_t mean = hint.nnz / A->rows;
        if (one_chunk) move();
        else if (mean < 10) launch(k_given_finish<256>, 256);
        else if (mean < 20) launch(k_given_finish<128>, 128);
        else if (mean < 40) launch(k_given_finish<64>, 64);
        else launch(k_given_finish<32>, 32);
    }
    phase_end(ctx, TSP_PHASE_NUMERIC, s);
    TSP_HIP_CHECK(ctx, hipGetLastError());
    const int rc = wait_published_scalars(ctx, ctx->publish_tag, s);
    if (rc) return rc;
    const int64_t *h = ctx->h_scalars;
    ctx->scalars_clean = ctx->arrivals_clean = !h[S_INTERNAL];       // (cleared for the next call)
    if (h[S_INVALID]) return TSP_ERR_NOT_CANONICAL;
    if (h[S_ROW_HEAVY] || h[S_INTERNAL]) {
        hint.given.missed();
        *end = kRowsAgain;
        return TSP_OK;
    }
    const int64_t nnz = h[S_C_NNZ];
    hint.candidates = h[S_CANDIDATES];
    hint.a_tiles = h[S_TILES_A];
    hint.products = h[S_ROW_PRODUCTS];
    hint.nnz = nnz;
    // (as k_row_prepare counts them; by 8 lanes there are none, or the product has been started again)
    hint.wide = h[S_ROW_WIDE] > A->rows / 64;
    hint.tiles = !rows_preferred(h[S_ROW_PRODUCTS], h[S_ROW_PRODUCTS], hint.wide ? 16 : cost_lanes, 0, true, h[S_CANDIDATES]);
    if (hint.tiles) {
        *end = kRowsNotTaken;
        return TSP_OK;
    }
    if (nnz > room) {
        copy.c_col = col = ws.get<int32_t>((size_t)nnz);
        copy.c_val = val = ws.get<float>((size_t)nnz);
        copy.live = nullptr;
        if (ws.failed) return TSP_ERR_ALLOC_FAILED;
        move();
        TSP_HIP_CHECK(ctx, hipGetLastError());
    }
    ctx->stats.a_tiles = h[S_TILES_A];
    ctx->stats.b_tiles = h[S_TILES_B];
    ctx->stats.candidate_pairs = h[S_CANDIDATES];
    ctx->stats.pairs = 0;
    ctx->stats.c_tiles = 0;
    ctx->stats.c_nnz = nnz;
    fill_selection_criteria(ctx, A->rows, A->nnz, h[S_TILES_A]);
    ws.keep(row_ptr);
    ws.keep(col);
    ws.keep(val);
    hint.given.taken();
    *C = tsp_csr{};
    C->rows = A->rows;
    C->cols = B->cols;
    C->nnz = nnz;
    C->row_ptr = row_ptr;
    C->col_idx = col;
    C->val = val;
    C->row_ptr_type = TSP_I64;
    C->val_type = TSP_F32;
    *end = kRowsTaken;
    return TSP_OK;
}

static int rowwise_run(tsp_context *ctx, const tsp_csr *A, const tsp_csr *B, bool alias, tsp_csr *C, hipStream_t s, RowsEnd *end,
                       RowHint **remembered) {
    *end = kRowsNotTaken;
    // Options that choose among the tile kernels, and shapes this path is not for: fewer rows than CUs (the sizing pass
    // has a block per heavy row), rows of more columns than the bitmaps of k_row_prepare hold (60 KB)
    if (!ctx->matrix_cores || ctx->numeric_run_len || ctx->work_order || ctx->strip_order || ctx->force_wide) return TSP_OK;
    int64_t most_cols = (int64_t)60 * 1024 * 8 * T;
    if (A->rows < 256 || A->rows > (1 << 27) || A->nnz == 0 || B->nnz == 0 || A->cols > most_cols || B->cols > most_cols) return TSP_OK;
    RowHint &hint = ctx->row_hints.find({{A->rows, A->nnz, B->rows, B->nnz, B->cols, alias}}, [](RowHint &) {});
    const bool known = hint.ready;
    if (known && hint.tiles) {
        *remembered = &hint;
        return TSP_OK;
    }
    if (A->nnz >= (1 << 28) || B->nnz >= (1 << 28)) return TSP_OK;      // (32-bit byte offsets into 8-byte records)
    const int64_t a_ntr = (A->rows + T - 1) / T, b_ntr = (B->rows + T - 1) / T;
    // Small rows: up to 24, 48, 96 or 192 products, with a margin over the mean number; for a row of B as many lanes as its mean has
    // entries.  For the row 8 lanes where the mean row of A has no more entries, else 16.  16 also
    // - for more than 32 products on average, for which 8 lanes sort 64 keys, eight to a lane (they have no more than 64): 65,536 and
    //   20,000 rows of 6 random entries, 36 products, 37.1 and 25.3 us of kernels by 8 lanes, 34.9 and 24.9 by 16; meshes, 25 products,
    //   300 x 300 25.9 and 29.2, 512 x 512 47.6 and 62.6; 65,536 rows of 3 entries 27.7 and 28.1;
    // - for few rows, whose rows of 9 to 16 entries are then no work for other kernels (where there are none 8 lanes take 1 us less of 13 to
    //   17 on meshes of 37, 80 and 110 squared, and the call as long as before);
    // - where more than one row in 64 is small but for its 9 to 16 entries (such a row costs 13 ns as a heavy one, and twice the
    //   lanes 0.1 ns per row; by the last product of these sizes, and where the one at hand turns out otherwise it is started
    //   again).
    // (Sums are rounded once whichever it is.)
    constexpr int64_t kFewRows = 12288;
    SmallShape shape{8, 1, 24};
    int lanes_unless_wide = 16, cost_lanes = 16;             // (rows_preferred's times are of 8 lanes for all of few entries)
    {
        const double list = (double)B->nnz / (double)std::max<int64_t>(B->rows, 1), mean = (double)A->nnz / (double)A->rows * list;
        while (shape.products < 192 && shape.products < 1.25 * mean) shape.products *= 2;
        if (A->nnz <= 8 * A->rows && shape.products <= 96) cost_lanes = 8;
        if (A->nnz <= 8 * A->rows && mean <= 32 && A->rows > kFewRows) lanes_unless_wide = 8;
        shape.lanes = known && hint.wide ? 16 : lanes_unless_wide;
        while (shape.list_lanes < shape.lanes && shape.list_lanes < list) shape.list_lanes *= 2;
    }
    // (16 GiB for the entries of the small rows at most: up to 89 million rows)
    auto found_entries = [&] { return ((A->rows * shape.lanes + 255) / 256) * 256 / shape.lanes * shape.products; };
    while (shape.products > 24 && found_entries() > kFoundEntries) shape.products /= 2;
    if (found_entries() > kFoundEntries) return TSP_OK;
    // straight from the operands, by the last product of these sizes.  Up to 128 entries per tile-row on average, the two trips of a wave
    // for which k_row_prepare gives it tile-rows as well; count_tiles would take more, which has not been timed.
    auto of_waves = [](const tsp_csr *M) { return M->nnz <= 128 * ((M->rows + T - 1) / T) && ((M->cols + T * 32 - 1) / (T * 32) + 3) / 4 * 64 <= (int64_t)kGivenBitmaps; };
    if (known && hint.nnz >= 0 && hint.heavy == 0 && hint.small && hint.given.allowed() && shape.lanes == lanes_unless_wide && A->rows <= kFinishRows &&
        (A->rows * shape.lanes + 255) / 256 <= kGivenBlocks && A->row_ptr_type == B->row_ptr_type && A->val_type == B->val_type && of_waves(A) && (alias || of_waves(B))) {
        const bool f16 = A->val_type == TSP_F16, i32 = A->row_ptr_type == TSP_I32;
        auto run = i32 ? (f16 ? rowwise_given<int32_t, uint16_t> : rowwise_given<int32_t, float>) : f16 ? rowwise_given<int64_t, uint16_t> : rowwise_given<int64_t, float>;
        return run(ctx, A, B, alias, C, s, hint, shape, cost_lanes, end);
    }
    const int64_t small_waves = ((A->rows * shape.lanes + 255) / 256) * 4;
    const int shift = B->cols <= 2048 ? 11 : 12;
    const int windows = (int)((B->cols + (1 << shift) - 1) >> shift);
    // heavy rows: the table of windows within 4 GiB, the arrays of B within the 32-bit byte offsets of stream_pieces
    const bool table_fits = (windows == 1 || B->rows * (windows + 1) * 4 <= (int64_t)4 << 30) && B->nnz < (1 << 28);

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
    const int64_t chunks = (A->rows + kChunkRows - 1) / kChunkRows;
    LeftOperand left{};
    left.ub = ws.get<int32_t>((size_t)A->rows);
    left.rows_of = ws.get<uint32_t>((size_t)a_ntr);
    left.products = ws.get<unsigned long long>((size_t)a_ntr);
    left.B = B;
    left.shape = shape;
    left.windows = windows;
    left.long_rows = known && hint.longest >= kLongRow;
    left.large_products = (int64_t)windows << shift <= kNarrowColumns ? kLargeNarrow : kLarge;
    unsigned long long *partial = ws.get<unsigned long long>((size_t)kPlanBlocks * kPlanSums);
    // (tasks of a product not seen before: one per heavy row and some more; where that is too few the lists are made again)
    left.heavy_cap = known ? hint.heavy : A->rows;
    left.task_cap = known ? hint.tasks : std::min<int64_t>(A->rows * (int64_t)windows, 2 * A->rows + 4096);
    left.heavy = ws.get<int32_t>((size_t)std::max<int64_t>(left.heavy_cap, 1));
    left.tasks = ws.get<int4>((size_t)std::max<int64_t>(left.task_cap, 1));
    int32_t *row_nnz = ws.get<int32_t>((size_t)A->rows + 1);
    uint32_t *group_len = ws.get<uint32_t>((size_t)chunks * kChunkTileRows);
    // a product of small rows only, by the last one of these sizes: k_small_finish
    const bool finish_and_copy = known && hint.nnz >= 0 && hint.heavy == 0 && hint.small && chunks > 1 && A->rows <= kFinishRows;
    if (finish_and_copy) left.part_len = ws.get<uint32_t>((size_t)((A->rows + kPartRows - 1) / kPartRows) * kPartStride);
    int2 *found = nullptr;
    int32_t *wave_total = nullptr, *live = nullptr, *only_small = nullptr;
    Expected expected{};
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;

    phase_begin(ctx, TSP_PHASE_CONVERT, s);
    const int64_t *skip = nullptr;
    if (!known && hint.sample && sample_pays(A->rows, A->nnz)) {
        skip = ctx->d_scalars + S_ROW_SKIP;
        SampleArgs a{};
        const tsp_csr *M[2] = {A, B};
        int64_t words = 0;
        for (int m = 0; m < 2; ++m) {
            a.row_ptr[m] = M[m]->row_ptr;
            a.col[m] = M[m]->col_idx;
            a.rows[m] = M[m]->rows;
            a.cols[m] = M[m]->cols;
            a.nnz[m] = M[m]->nnz;
            a.is_i64[m] = M[m]->row_ptr_type == TSP_I64;
            a.blocks[m] = m && alias ? 0 : (int)std::min<int64_t>(kSampleRows, m ? b_ntr : a_ntr);
            words = std::max(words, (M[m]->cols + T * 32 - 1) / (T * 32));
        }
        a.small_lanes = known && hint.wide ? 16 : cost_lanes;
        a.small_products = shape.products;
        a.d_scalars = ctx->d_scalars;
        hipLaunchKernelGGL(k_row_sample, dim3((unsigned)(a.blocks[0] + a.blocks[1])), dim3(256), (size_t)words * 4, s, a);
    }
    {
        KernelTimer kt(ctx, TSP_KERNEL_CONVERT, s);
        prepare(ctx, A, ma, left, alias ? nullptr : B, mb, s, skip);
    }
    phase_end(ctx, TSP_PHASE_CONVERT, s);
    TSP_HIP_CHECK(ctx, hipGetLastError());

    SumArgs sums{};
    sums.a_tile_rows = a_ntr;
    sums.b_tile_rows = b_ntr;
    sums.a_start = ma.start;
    sums.a_ntiles = ma.ntiles;
    sums.a_tile_col = ma.tile_col;
    sums.b_ntiles = mb.ntiles;
    sums.rows_of = left.rows_of;
    sums.a_range = ma.range;
    sums.b_range = mb.range;
    sums.products = left.products;
    sums.same = alias;
    sums.partial = partial;
    sums.skip = skip;
    // (a tile-row to a wave, whose tiles are more than a group of lanes takes; for the smallest products as few blocks as do)
    const int per_block = chunks == 1 ? 16 : 4;
    const int sum_blocks = (int)std::min<int64_t>(kPlanBlocks, (std::max(a_ntr, alias ? 0 : b_ntr) + per_block - 1) / per_block);
    // row_ptr of C when the sizes of its rows are there, and the sizes of everything to the host
    int64_t *row_ptr = nullptr;
    auto finish_args = [&] {
        FinishArgs a{};
        a.partial = partial;
        a.partials = sum_blocks;
        a.same = alias;
        a.d_scalars = ctx->d_scalars;
        a.h_scalars_dev = ctx->h_scalars_dev;
        a.clear = row_ptr != nullptr;
        a.expected = expected;
        a.live = live;
        a.skip = skip;
        if (row_ptr && A->rows <= kFinishRows) {
            a.rows = A->rows;
            a.row_nnz = row_nnz;
            a.group_len = group_len;
            a.c_row_ptr = row_ptr;
        }
        a.publish_tag = ++ctx->publish_tag;
        return a;
    };
    auto finish = [&](int timer) {
        KernelTimer kt(ctx, timer, s);
        unsigned blocks = 1;
        if (!row_ptr) {
            hipLaunchKernelGGL(k_row_sums, dim3((unsigned)sum_blocks), dim3(256), 0, s, sums);
        } else if (A->rows <= kFinishRows) {
            blocks = (unsigned)chunks;
        } else {
            int64_t *tmp = ws.get<int64_t>(scan_tmp_entries(A->rows));
            if (!tmp) return (int)TSP_ERR_ALLOC_FAILED;
            const int rc = scan_exclusive_i32_to_i64(ctx, row_nnz, row_ptr, A->rows, ctx->d_scalars + S_C_NNZ, nullptr, tmp, s);
            if (rc) return rc;
        }
        hipLaunchKernelGGL(k_row_finish, dim3(blocks), dim3(256), 0, s, finish_args());
        TSP_HIP_CHECK(ctx, hipGetLastError());
        return (int)TSP_OK;
    };
    int64_t n_heavy = left.heavy_cap, n_tasks = left.task_cap, n_large = known ? hint.large_tasks : 0, n_products = known ? hint.products : 0;
    FillKind kind{};
    bool other_lanes = false;                // the product at hand wants its small rows by another number of lanes
    auto sizes_known = [&]() {               // the host has the numbers of k_row_finish
        const int64_t *h = ctx->h_scalars;
        if (h[S_INVALID]) return (int)TSP_ERR_NOT_CANONICAL;
        n_heavy = h[S_ROW_HEAVY];
        n_tasks = h[S_ROW_TASKS];
        n_large = h[S_ROW_LARGE_TASKS];
        n_products = h[S_ROW_PRODUCTS];
        hint.ready = true;
        hint.wide = h[S_ROW_WIDE] > A->rows / 64;
        other_lanes = shape.lanes != (hint.wide ? 16 : lanes_unless_wide);
        const int64_t heavy = shape.lanes == 8 && hint.wide ? n_heavy - std::min(n_heavy, h[S_ROW_WIDE]) : n_heavy;
        const int64_t small = std::min(h[S_ROW_PRODUCTS], (A->rows - heavy) * shape.products);      // (at most)
        kind = fill_kind(h);
        hint.tiles = !rows_preferred(h[S_ROW_PRODUCTS], small, hint.wide ? 16 : cost_lanes, heavy, kind.sum != FillKind::kDouble, h[S_CANDIDATES]) ||
                      (n_heavy > 0 && !table_fits) || n_tasks >= INT32_MAX;
        hint.candidates = h[S_CANDIDATES];
        hint.a_tiles = h[S_TILES_A];
        hint.heavy = n_heavy;
        hint.given.other_way(n_heavy == 0);
        hint.tasks = n_tasks;
        hint.large_tasks = n_large;
        hint.products = n_products;
        hint.longest = h[S_ROW_LONGEST];
        hint.small = h[S_ROW_SMALL] > 0;
        hint.nnz = row_ptr ? h[S_C_NNZ] : -1;
        hint.sum = kind.sum;
        hint.scale = kind.scale;
        return (int)TSP_OK;
    };
    if (!known) {
        int rc = finish(TSP_KERNEL_SCAN_SYM);
        if (!rc) rc = wait_published_scalars(ctx, ctx->publish_tag, s);
        if (!rc && skip && ctx->h_scalars[S_ROW_SKIP]) {
            hint.ready = hint.tiles = hint.estimated = true;
            hint.candidates = ctx->h_scalars[S_ROW_SKIP] - 1;
            *remembered = &hint;
            return TSP_OK;
        }
        sums.skip = skip = nullptr;
        if (!rc) rc = sizes_known();
        if (rc) return rc;
        if (hint.tiles || other_lanes) {     // (the tile kernels start over; the scalars they use are cleared for them)
            *end = hint.tiles ? kRowsNotTaken : kRowsAgain;
            return TSP_OK;
        }
    }

    phase_begin(ctx, TSP_PHASE_SYMBOLIC, s);
    row_ptr = ws.get<int64_t>((size_t)A->rows + 1);
    found = ws.get<int2>((size_t)found_entries());
    wave_total = ws.get<int32_t>((size_t)small_waves);
    if (ws.failed) return TSP_ERR_ALLOC_FAILED;
    uint32_t *pack = nullptr, *offset = nullptr, *bits = nullptr;
    int64_t bit_rows = 0;                    // rows whose pattern `bits` holds
    bool pattern_kept = false;               // ... and the sizing pass has left that of all heavy rows there
    CountArgs c{};
    auto count_heavy = [&](int64_t rows, int64_t large) {    // the large ones apart from the others, or all of them alike
        const size_t lds = ((size_t)c.span_windows << (shift - 3)) + 256;
        c.n_large = large;
        c.large_products = large > 0 ? left.large_products : 0;
        if (large > 0) {
            auto kernel = shift == 11 ? k_heavy_count<2048, 1024, true> : k_heavy_count<4096, 1024, true>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)large), dim3(1024), lds, s, c);
        }
        const bool wide = c.span_windows > kSpanWindows / 2;
        auto kernel = shift == 11 ? k_heavy_count<2048, kCountThreads, false>
                      : wide      ? k_heavy_count<4096, kCountThreadsWide, false> : k_heavy_count<4096, kCountThreads, false>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)rows), dim3(wide ? kCountThreadsWide : kCountThreads), lds, s, c);
    };
    // heavy rows whose pattern is kept at a time
    auto pattern_rows = [&](int64_t heavy) { return std::min(heavy, std::max<int64_t>(ctx->pattern_bytes / (((int64_t)windows << shift) / 8), 1)); };
    int32_t *table = nullptr, *words = nullptr;
    uint32_t *word = nullptr;
    int32_t *span_table = nullptr;
    const int spans = (windows + kSpanWindows - 1) / kSpanWindows;
    SmallArgs m{};
    m.shape = shape;
    m.rows = A->rows;
    const PreparedOperands prepared{ma.start, mb.start, left.ub, ma.rec, mb.rec};
    m.wave_bytes = (int)shape.wave_bytes();
    m.found = found;
    m.wave_total = wave_total;
    m.row_nnz = row_nnz;
    m.group_len = group_len;
    const unsigned small_blocks = (unsigned)(small_waves / 4);
    m.sum_blocks = sum_blocks;
    m.sums_first = std::max(a_ntr, alias ? 0 : b_ntr) > 16 * kPlanBlocks;
    // (a small product without heavy rows: the last block of the small ones finishes)
    bool finish_too = known && hint.nnz >= 0 && chunks == 1 && n_heavy == 0;
    auto heavy_arrays = [&]() {
        if (n_heavy == 0) return (int)TSP_OK;
        if (!pack) {
            pack = ws.get<uint32_t>((size_t)B->nnz + 64);     // (a piece is read whole)
            word = ws.get<uint32_t>((size_t)B->nnz + 64);
            if (spans > 1) span_table = ws.get<int32_t>((size_t)B->rows * (spans + 1));
            words = ws.get<int32_t>((size_t)B->rows);
            if (windows > 1) table = ws.get<int32_t>((size_t)B->rows * (windows + 1));
        }
        offset = ws.get<uint32_t>((size_t)n_heavy * windows);
        // the pattern of the heavy rows, kept for the multiplication: a bit per column, also of the empty windows.
        // Where that is too much, the multiplication has it found again, some rows at a time.
        const int64_t row_words = ((int64_t)windows << shift) / 32;
        bit_rows = pattern_rows(n_heavy);
        while (!(bits = ws.get_if_there<uint32_t>((size_t)(bit_rows * row_words))) && bit_rows > 1) bit_rows /= 2;
        return ws.failed || !bits ? (int)TSP_ERR_ALLOC_FAILED : (int)TSP_OK;
    };
    auto size_rows = [&](bool again) {
        if (again || n_tasks > left.task_cap || n_heavy > left.heavy_cap) {
            // the lists did not fit: make them again, as large as they have to be
            left.heavy_cap = n_heavy;
            left.task_cap = n_tasks;
            left.heavy = ws.get<int32_t>((size_t)std::max<int64_t>(n_heavy, 1));
            left.tasks = ws.get<int4>((size_t)std::max<int64_t>(n_tasks, 1));
            if (ws.failed) return (int)TSP_ERR_ALLOC_FAILED;
            hipLaunchKernelGGL(k_clear_lists, dim3(1), dim3(64), 0, s, ctx->d_scalars);
            prepare(ctx, A, ma, left, nullptr, mb, s, nullptr);
            if (again) {
                const int rc = heavy_arrays();
                if (rc) return rc;
            }
        }
        KernelTimer kt(ctx, TSP_KERNEL_SYM_COUNT, s);
        m.finish = finish_too;
        auto launch = [&](auto kernel, const auto &p, unsigned pack_blocks) {
            hipLaunchKernelGGL(kernel, dim3(pack_blocks + small_blocks + (unsigned)sum_blocks), dim3(256), 4 * shape.wave_bytes() + SmallShape::kReadPast, s, m, prepared, sums,
                               finish_too ? finish_args() : FinishArgs{}, p);
        };
        const bool at_once = n_heavy > 0 && B->rows <= kPackRows;
        PackArgs p{B->rows, mb.start, mb.rec, pack, word, words, table, span_table, windows, spans, shift, 0, 0, 0};
        // (a wave per row where the mean row fills it; for all of them the products of R-MAT graphs of scale 10 to 16 take 1 to 5 %
        // longer: 12 87.4 -> 91.5 us, 14 274 -> 280, 16 2235 -> 2255)
        p.lanes = B->nnz > 64 * B->rows ? 64 : 16;
        p.medium_from = pack_short(p.lanes) + 1;
        p.blocks = kLongBlocks + (uint32_t)((B->rows * p.lanes + (at_once ? 255 : kPackThreads - 1)) / (at_once ? 256 : kPackThreads));
        auto small_rows = [&](auto pack, unsigned pack_blocks) {
            using Pack = decltype(pack);
            if (shape.lanes == 8) launch(shape.narrow() ? k_row_small<8, true, Pack> : k_row_small<8, false, Pack>, pack, pack_blocks);
            else launch(shape.narrow() ? k_row_small<16, true, Pack> : k_row_small<16, false, Pack>, pack, pack_blocks);
        };
        if (at_once) small_rows(p, p.blocks);
        else small_rows(NoPack{}, 0);
        if (n_heavy > 0) {
            if (!at_once) hipLaunchKernelGGL(k_heavy_pack, dim3(p.blocks), dim3(kPackThreads), 0, s, p);
            c.heavy = left.heavy;
            c.heavy_cap = n_heavy;
            c.d_scalars = ctx->d_scalars;
            c.a_start = ma.start;
            c.b_start = mb.start;
            c.a_rec = ma.rec;
            c.b_word = word;
            c.b_words = words;
            c.b_spans = span_table;
            c.b_nnz = (int32_t)B->nnz;
            c.spans = spans;
            c.windows = windows;
            c.span_windows = std::min(windows, kSpanWindows);
            c.row_nnz = row_nnz;
            c.group_len = group_len;
            c.offset = offset;
            pattern_kept = bit_rows == n_heavy;
            c.bits = pattern_kept ? bits : nullptr;
            c.tasks = left.tasks;
            c.ub = left.ub;
            count_heavy(n_heavy, n_products >= kSplitProducts ? n_large : 0);
        }
        return (int)TSP_OK;
    };
    int32_t *col = nullptr;
    float *val = nullptr;
    auto multiply = [&](bool small, FillKind how) {
        phase_begin(ctx, TSP_PHASE_NUMERIC, s);
        KernelTimer kt(ctx, TSP_KERNEL_NUMERIC, s);
        if (small) {
            const CopyArgs p{shape, A->rows, small_waves, ma.start, left.ub, found, wave_total, row_ptr, col, val, live};
            hipLaunchKernelGGL(k_small_copy, dim3(small_blocks), dim3(256), 0, s, p);
        }
        if (n_tasks > 0) {
            FillArgs f{};
            f.tasks = left.tasks;
            f.n_tasks = n_tasks;
            f.n_large = n_large;
            f.task_cap = left.task_cap;
            f.a_start = ma.start;
            f.b_start = mb.start;
            f.a_rec = ma.rec;
            f.pack = pack;
            f.table = table;
            f.b_nnz = (int32_t)B->nnz;
            f.windows = windows;
            f.offset = offset;
            f.bits = bits;
            f.c_row_ptr = row_ptr;
            f.c_col = col;
            f.c_val = val;
            f.live = live;
            f.window_shift = shift;
            for (int64_t from = 0; from < n_heavy; from += bit_rows) {
                f.heavy_from = (int)from;
                f.heavy_to = (int)std::min(from + bit_rows, n_heavy);
                // (by what the sizing pass did: it went by the heavy rows of the last product, which may have been more)
                if (!pattern_kept) {
                    c.d_scalars = nullptr;
                    c.row_nnz = nullptr;
                    c.heavy_cap = f.heavy_to;
                    c.heavy_from = f.heavy_from;
                    c.bits = bits;
                    count_heavy(f.heavy_to - f.heavy_from, 0);
                }
                launch_fill(f, how, B->nnz <= 16 * B->rows, n_products >= kSplitProducts, s);
            }
        }
        phase_end(ctx, TSP_PHASE_NUMERIC, s);
        TSP_HIP_CHECK(ctx, hipGetLastError());
        return (int)TSP_OK;
    };
    // A product of the sizes of the last one: the kernels of the multiplication follow at once, into arrays for as many
    // entries as that one had and some more, and k_row_finish lets them run if this product fits; the GPU does not
    // wait for the host to learn nnz(C) (8 us of 78 on a 512x512 mesh).  Otherwise they are launched again below.
    int rc = heavy_arrays();
    if (rc) return rc;
    const bool ahead = known && hint.nnz >= 0 && bit_rows == n_heavy;
    int64_t room = 0;
    if (ahead) {
        room = hint.nnz + std::min<int64_t>(hint.nnz / 16, 1 << 20);
        col = ws.get<int32_t>((size_t)room);
        val = ws.get<float>((size_t)room);
        live = ws.get<int32_t>(3);
        if (ws.failed) return TSP_ERR_ALLOC_FAILED;
        kind = FillKind{(FillKind::Sum)hint.sum, hint.scale};
        expected = Expected{room, n_heavy, n_tasks, n_large, kind};
    }
    const bool had_small = hint.small;
    if (finish_and_copy) {
        only_small = ws.get<int32_t>(1);
        if (!only_small) return TSP_ERR_ALLOC_FAILED;
        m.part_len = left.part_len;
        m.only_small = only_small;
        m.d_scalars = ctx->d_scalars;
    }
    rc = size_rows(false);
    if (rc) return rc;
    phase_end(ctx, TSP_PHASE_SYMBOLIC, s);
    // (row_ptr and the entries by one kernel: it counts as the multiplication)
    const auto finish_phase = finish_and_copy ? TSP_PHASE_NUMERIC : TSP_PHASE_COUNT;
    phase_begin(ctx, finish_phase, s);
    if (finish_and_copy) {
        KernelTimer kt(ctx, TSP_KERNEL_NUMERIC, s);
        FinishArgs a = finish_args();
        a.live = nullptr;
        const CopyArgs p{shape, A->rows, small_waves, ma.start, left.ub, found, wave_total, row_ptr, col, val, nullptr};
        auto launch = [&](auto kernel, int rows) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((A->rows + rows - 1) / rows)), dim3(256), 0, s, a, p, left.part_len, only_small);
        };
        // (about 2000 entries to a block: a 512 x 512 mesh 13.5 / 12.4 / 15.4 us with 256 / 128 / 64 rows, 65,536 rows of 60 entries
        // 17.7 / 13.6 / 12.4 / 15.5 with 128 / 64 / 32 / 16, A*P on a 64^3 grid 7.6 / 8.8 / 12.4 with 256 / 128 / 64)
        const int64_t mean = hint.nnz / A->rows;
        if (mean < 10) launch(k_small_finish<256>, 256);
        else if (mean < 20) launch(k_small_finish<128>, 128);
        else if (mean < 40) launch(k_small_finish<64>, 64);
        else launch(k_small_finish<32>, 32);
        TSP_HIP_CHECK(ctx, hipGetLastError());
    } else if (!finish_too) {
        rc = finish(TSP_KERNEL_SCAN_ROWS);
    }
    ctx->scalars_clean = !rc;                // (it has cleared the scalar block for the next call)
    phase_end(ctx, finish_phase, s);
    if (!rc && ahead && !finish_and_copy) rc = multiply(had_small, kind);
    if (!rc) rc = wait_published_scalars(ctx, ctx->publish_tag, s);           // the wait that sizes C
    if (rc) return rc;
    const int64_t had_heavy = n_heavy, had_tasks = n_tasks, had_large = n_large, products = ctx->h_scalars[S_PRODUCTS];
    rc = sizes_known();
    if (rc) return rc;
    if (hint.tiles || other_lanes) {         // another matrix of the same sizes: as it would be done if it had come first
        *end = hint.tiles ? kRowsNotTaken : kRowsAgain;
        return TSP_OK;
    }
    const bool done = ahead && expected.holds(ctx->h_scalars) && (had_small || ctx->h_scalars[S_ROW_SMALL] == 0);
    if (!done) {
        live = nullptr;
        if (n_heavy > had_heavy || n_tasks > had_tasks || n_large > had_large) {            // another matrix of the same sizes, with more work in it
            ctx->scalars_clean = finish_too = false;
            rc = size_rows(true);
            if (rc) return rc;
            rc = finish(TSP_KERNEL_SCAN_ROWS);
            ctx->scalars_clean = !rc;
            if (!rc) rc = wait_published_scalars(ctx, ctx->publish_tag, s);
            if (rc) return rc;
            ctx->h_scalars[S_PRODUCTS] = products;
            hint.nnz = ctx->h_scalars[S_C_NNZ];
        }
        if (ctx->h_scalars[S_C_NNZ] > room || !ahead) {
            col = ws.get<int32_t>((size_t)ctx->h_scalars[S_C_NNZ]);
            val = ws.get<float>((size_t)ctx->h_scalars[S_C_NNZ]);
            if (ws.failed) return TSP_ERR_ALLOC_FAILED;
        }
        if (ctx->h_scalars[S_C_NNZ] > 0) rc = multiply(ctx->h_scalars[S_ROW_SMALL] > 0, kind);
        if (rc) return rc;
    }
    const int64_t nnz = ctx->h_scalars[S_C_NNZ];
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
    *end = kRowsTaken;
    return TSP_OK;
}

// What has been learnt of a product decides how the next one of the same sizes is started, and not how its entries are
// summed: where the product at hand asks for another number of lanes or for tiles it is started again.  So a product has
// the same bits as often as it is repeated.
int rowwise_spgemm(tsp_context *ctx, const tsp_csr *A, const tsp_csr *B, bool alias, tsp_csr *C, hipStream_t s, bool *taken,
                   RowHint **remembered) {
    *remembered = nullptr;
    RowsEnd end = kRowsNotTaken;
    int rc = TSP_OK;
    for (int runs = 0; runs < 3; ++runs) {                   // (straight from the operands, by 8 lanes, by 16)
        const int64_t tag = ctx->publish_tag;
        rc = rowwise_run(ctx, A, B, alias, C, s, &end, remembered);
        if (rc || end == kRowsTaken) break;
        if (ctx->publish_tag != tag) {
            hipLaunchKernelGGL(k_clear_rows, dim3(1), dim3(64), 0, s, ctx->d_scalars, ctx->h_scalars[S_PRODUCTS]);
            ctx->scalars_clean = false;
        }
        if (end != kRowsAgain) break;
    }
    *taken = end == kRowsTaken;
    return rc;
}

}  // namespace tsp
