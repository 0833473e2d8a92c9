// Compaction of zeros (paper Section 4.4; the two compaction steps that end Algorithm 1): the multiplication pass writes
// every structural position of C; numerical cancellation (and stored zeros in the inputs) leaves
// some of them with the value 0.  This pass removes them, so that the result is strictly sparse:
// count the survivors, prefix-sum, copy the survivors in order.
// The paper compacts the element array with a library primitive and drops empty tiles; here the
// output is already CSR.
//
// All three passes go by the entries and not by the rows, so that rows of any length weigh the same: a block takes a
// chunk of 4096 consecutive entries (a multiple of that on very large matrices) and finds the rows that begin in it by a
// search in row_ptr.  Bound by memory: the values twice, the columns once, the survivors.  200,003 rows of 60 entries on
// average, a fifth zero: count 8.7 us, copy 31 us, the sums in it (with a launch of their own 8.7 + 4.6 + 30).  One pass that reads the
// values once and waits for the sums of the blocks before takes 39: of blocks that all load, then all wait, then all write.
// Only the entries between the first and the last row pointer are C's.  A block finds the new pointers of the first 4096 rows
// that begin in its part; where there are more (empty ones, then), blocks for 4096 rows each find the others (300,000 rows
// of 2000 entries 37 us for the call, 663 with all rows of a part left to its block; 81 by rows).
//
// The searches need row pointers that do not go down.  The counting pass looks, and where they do (no CSR matrix, but none
// that is refused) the pass is made again with every pointer replaced by the largest so far.
#include "common.hpp"

#include <algorithm>
#include <mutex>

namespace tsp {

constexpr int kCompactThreads = 256;
constexpr int kCompactPart = 4096;             // entries a block holds at a time, 16 per thread
constexpr int64_t kCompactChunks = 65536;      // at most
// Up to so many blocks of the counting pass the copying blocks add up the counts before theirs themselves (a block reads two bytes for every
// one), and the host gets the total from one of them that does nothing else; beyond, one block makes all the sums, in a launch of its
// own (200,003 rows of 60 entries, 3126 blocks: 4.6 us and the gap before it).
constexpr int64_t kCompactSums = 16384;
constexpr int kCheckRows = 1024;               // rows per block that looks whether row pointers ascend
constexpr int kCompactRows = 4096;             // rows whose new pointers a part's block finds, and rows of a block of their own

template <typename RP>
struct CompactArgs {
    const RP *row_ptr;
    const int32_t *col;
    const float *val;
    int64_t rows, nnz;                         // (rows: -1 where only columns and values are wanted)
    int64_t last;                              // index of the last row pointer
    int64_t chunk;                             // entries per block, a multiple of kCompactPart
    int chunks;
    // Counts of the blocks of the counting pass (those of rows first) to be added up, with what they have found in the two upper bits; or
    // null: `before` has the sums.
    const uint16_t *counts;
    int64_t capacity;                          // of the result's columns and values
    // Not 0 where nothing is to be copied unless an entry is dropped: what before[chunks] then holds, from the blocks of the counting pass
    // that drop one (with `counts`; never the same twice on a handle, so the word needs no other value before)
    int64_t mark;
    // blocks for `per` rows each; they come before the chunks' in a launch (behind them they would end it)
    __host__ __device__ int row_blocks(int per) const { return rows < 0 ? 0 : (int)(rows / per) + 1; }
};
template <typename RP>
__device__ __forceinline__ int64_t clamped(const CompactArgs<RP> &a, int64_t row) {
    return min(max((int64_t)a.row_ptr[row], (int64_t)0), a.nnz);
}
// The entries of the matrix.  (A part is loaded without waiting for these: those outside count as zeros.)
struct EntryRange {
    int64_t lo, hi;
};
template <typename RP>
__device__ __forceinline__ EntryRange entry_range(const CompactArgs<RP> &a) {
    return {min(max((int64_t)uniform_load(a.row_ptr), (int64_t)0), a.nnz),
            min(max((int64_t)uniform_load(a.row_ptr + a.last), (int64_t)0), a.nnz)};
}
__device__ __forceinline__ void drop_outside(const EntryRange &range, int64_t begin, float (&v)[16]) {
    if (begin >= range.lo && begin + kCompactPart <= range.hi) return;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int64_t e = begin + u * kCompactThreads + threadIdx.x;
        v[u] = e >= range.lo && e < range.hi ? v[u] : 0.0f;
    }
}

// entries per chunk so that at most kCompactChunks cover nnz
static int64_t compact_chunk(int64_t nnz) {
    const int64_t parts = (nnz + kCompactPart - 1) / kCompactPart;
    return kCompactPart * std::max<int64_t>((parts + kCompactChunks - 1) / kCompactChunks, 1);
}
static int64_t compact_chunks(int64_t nnz) { return std::max<int64_t>((nnz + compact_chunk(nnz) - 1) / compact_chunk(nnz), 1); }

// +0.0 and -0.0 are zeros, NaN is not
__device__ __forceinline__ bool survives(float v) { return !(v == 0.0f); }

// The elements of the block's part of 4096, 16 per thread, 256 neighbours per load; zeros past the end.
template <typename X>
__device__ __forceinline__ void load_part(const X *from, int64_t begin, int64_t end, X (&x)[16]) {
    if (begin + kCompactPart <= end) {
        from += begin;
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = from[(unsigned)(u * kCompactThreads + threadIdx.x)];
        return;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int64_t e = begin + u * kCompactThreads + threadIdx.x;
        x[u] = e < end ? from[e] : X(0);
    }
}

// Survivors per chunk, and where the entries begin and end (before[chunks + 1], before[chunks + 2]); the blocks of the rows, whose
// counts come first, look
// whether the row pointers ascend, and whether more than kCompactRows rows may begin in one part.
template <typename RP>
__global__ __launch_bounds__(kCompactThreads) void k_compact_count(CompactArgs<RP> a, uint32_t *__restrict__ count,
                                                                   int64_t *__restrict__ before, int64_t *d_scalars) {
    __shared__ uint32_t s_wave[kCompactThreads / 64];
    const int b = (int)blockIdx.x - a.row_blocks(kCheckRows);
    if (b < 0) {
        bool down = false;
#pragma unroll
        for (int u = 0; u < kCheckRows / kCompactThreads; ++u) {
            const int64_t r = (int64_t)blockIdx.x * kCheckRows + u * kCompactThreads + threadIdx.x;
            down |= clamped(a, min(r, a.last)) > clamped(a, min(r + 1, a.last));
        }
        bool runs = false;
        // (such rows have the first row of some block among them, and 3072 behind it)
        if (threadIdx.x == 0) {
            const int64_t r = (int64_t)blockIdx.x * kCheckRows, last = min(r + kCompactRows - kCheckRows, a.last);
            auto part = [&](int64_t row) { return min(clamped(a, row), max(a.nnz - 1, (int64_t)0)) / kCompactPart; };
            runs = r < a.last && part(r) == part(last);
        }
        const int any_down = __syncthreads_or(down);
        if (a.counts) {
            if (threadIdx.x == 0) reinterpret_cast<uint16_t *>(count)[blockIdx.x] = (uint16_t)((any_down ? 1u << 14 : 0u) | (runs ? 1u << 15 : 0u));
        } else {
            if (any_down && threadIdx.x == 0) d_scalars[S_DESCENDS] = 1;
            if (runs) d_scalars[S_EMPTY_RUNS] = 1;
        }
        return;
    }
    const int64_t c0 = (int64_t)b * a.chunk, c1 = min(c0 + a.chunk, a.nnz);
    const EntryRange range = entry_range(a);
    if (b == 0 && threadIdx.x == 0) {
        before[a.chunks + 1] = range.lo;
        before[a.chunks + 2] = range.hi;
    }
    uint32_t n = 0;
    for (int64_t begin = c0; begin < c1; begin += kCompactPart) {
        float v[16];
        load_part(a.val, begin, c1, v);
        drop_outside(range, begin, v);
#pragma unroll
        for (int u = 0; u < 16; ++u) n += survives(v[u]) ? 1u : 0u;
    }
    n = wave_sum(n);
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t all = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        if (a.counts) reinterpret_cast<uint16_t *>(count)[blockIdx.x] = (uint16_t)all;
        else count[b] = all;
        if (a.mark && all < c1 - c0) before[a.chunks] = a.mark;
    }
}

// The sum of the first n counts, and what was found, by the whole block (two barriers)
struct CountSum {
    int64_t survivors;
    int found;                                 // 1: row pointers go down, 2: long runs of empty rows
};
__device__ __forceinline__ CountSum sum_counts(const uint16_t *counts, int n, uint32_t *s_wave, uint32_t *s_found) {
    uint32_t sum = 0, found = 0;
    const uint4 *const eights = reinterpret_cast<const uint4 *>(counts);
    const int whole = (n + 7) / 8;
    for (int q = threadIdx.x; q < whole; q += 2 * kCompactThreads) {
        uint4 x[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) x[u] = eights[min(q + u * kCompactThreads, whole - 1)];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t y[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
            const int left = n - (q + u * kCompactThreads) * 8;      // counts of these that are to be added up
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t two = left >= 2 * k + 2 ? y[k] : left > 2 * k ? y[k] & 0xFFFFu : 0u;
                sum += (two & 0x3FFFu) + (two >> 16 & 0x3FFFu);
                found |= two;
            }
        }
    }
    found = (found | found >> 16) >> 14 & 3u;
    sum = wave_sum(sum);                       // (fewer than 2^31 entries)
    found = (__any(found & 1u) ? 1u : 0u) | (__any(found & 2u) ? 2u : 0u);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s_wave[threadIdx.x >> 6] = sum;
        s_found[threadIdx.x >> 6] = found;
    }
    __syncthreads();
    return {(int64_t)s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3], (int)(s_found[0] | s_found[1] | s_found[2] | s_found[3])};
}

// Survivors before every chunk, by one block, 4096 chunks at a time; the total to the host.  (At most 65,536 numbers.)
// before[chunks]: 1 where the row pointers go down, 2 where there are long runs of empty rows.  The scalar block is left as it was.
__global__ __launch_bounds__(1024) void k_compact_scan(const uint32_t *__restrict__ count, int chunks, int64_t *__restrict__ before,
                                                      int64_t *d_scalars, int64_t *h_scalars_dev, int64_t publish_tag) {
    __shared__ uint64_t lds[1024 / 64];
    __shared__ int64_t own[kScalars];
    const int64_t standing = standing_scalar(d_scalars);
    uint64_t carry = 0;
    for (int t0 = 0; t0 < chunks; t0 += 4096) {
        const int first = t0 + (int)threadIdx.x * 4;
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = first + i < chunks ? count[first + i] : 0u;
        uint64_t total;
        uint64_t run = carry + block_exclusive_scan64<1024>((uint64_t)x[0] + x[1] + x[2] + x[3], &total, lds);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (first + i < chunks) before[first + i] = (int64_t)run;
            run += x[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) own[S_C_NNZ] = (int64_t)carry;
    const int64_t runs = __shfl(standing, S_EMPTY_RUNS, 64);
    if (threadIdx.x == S_DESCENDS) before[chunks] = standing | runs << 1;
    publish_scalars(d_scalars, h_scalars_dev, publish_tag, standing, own, own_slot(S_C_NNZ));
    if (threadIdx.x == S_C_NNZ || threadIdx.x == S_DESCENDS || threadIdx.x == S_EMPTY_RUNS) d_scalars[threadIdx.x] = 0;
}

// First row whose entries begin at `begin` or later (rows: none), by the 64 lanes of a wave.
template <typename RP>
__device__ __forceinline__ int64_t first_row_from(const RP *row_ptr, int64_t rows, int64_t begin) {
    int64_t lo = 0, hi = rows;                 // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + 63) / 64, at = lo + step * lane_id();
        const bool before = at < hi && max((int64_t)row_ptr[at], (int64_t)0) < begin;
        const int n = __popcll(__ballot(before));        // (the answer lies behind the n-th probe)
        if (n == 0) return lo;
        const int64_t base = lo;
        lo = base + step * (n - 1) + 1;
        hi = min(hi, base + step * n);
    }
    return lo;
}

// The survivors of the part at `begin`: lane l of every wave gets those of the part's 64-entry word l, and returns how many
// there are in the words before it.  (s_mask: as many words; a barrier before it is written again.)
__device__ __forceinline__ uint32_t part_words(const float (&v)[16], unsigned long long *s_mask, unsigned long long *word, uint32_t *all) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const unsigned long long m = __ballot(survives(v[u]));
        if (lane == 0) s_mask[u * (kCompactThreads / 64) + wave] = m;
    }
    __syncthreads();
    *word = s_mask[lane];
    const uint32_t n = (uint32_t)__popcll(*word), inc = wave_inclusive_scan(n);
    *all = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    return inc - n;
}
// ... and how many of them lie before entry `offset` of the part; all lanes take part
__device__ __forceinline__ int survivors_before(int offset, unsigned long long word, uint32_t prefix) {
    const int w = offset >> 6, words_before = __shfl((int)prefix, min(w, 63), 64);
    const unsigned long long own = __shfl(word, min(w, 63), 64);
    return words_before + (w < 64 ? __popcll(own & ((1ull << (offset & 63)) - 1ull)) : __popcll(own));
}

template <typename RP>
__global__ __launch_bounds__(kCompactThreads) void k_compact_fill(CompactArgs<RP> a, const int64_t *__restrict__ before,
                                                                 int64_t *__restrict__ new_row_ptr,
                                                                 int32_t *__restrict__ out_col,
                                                                 float *__restrict__ out_val, int64_t *d_scalars,
                                                                 int64_t *h_scalars_dev, int64_t publish_tag) {
    __shared__ unsigned long long s_mask[kCompactPart / 64];
    __shared__ uint32_t s_wave[kCompactThreads / 64], s_found[kCompactThreads / 64];
    const int checks = a.counts ? a.row_blocks(kCheckRows) : 0, teller = a.counts ? 1 : 0;
    if (teller && blockIdx.x == 0) {           // (the scalar block stays as it is)
        __shared__ int64_t own[kScalars];
        if (!publish_tag) return;
        const int64_t standing = standing_scalar(d_scalars);
        const CountSum all = sum_counts(a.counts, checks + a.chunks, s_wave, s_found);
        if (threadIdx.x < kScalars)
            own[threadIdx.x] = threadIdx.x == S_C_NNZ ? all.survivors : threadIdx.x == S_DESCENDS ? (all.found & 1) : threadIdx.x == S_EMPTY_RUNS ? 0 : standing;
        publish_mirror(h_scalars_dev, publish_tag, own);
        return;
    }
    if (a.mark && uniform_load(before + a.chunks) != a.mark) return;
    const EntryRange range{uniform_load(before + a.chunks + 1), uniform_load(before + a.chunks + 2)};
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int b = (int)blockIdx.x - teller - a.row_blocks(kCompactRows);
    if (b < 0) {
        // (where the row pointers go down nothing is written, and the host makes the pass again, see compact_descending)
        const int64_t found = a.counts ? sum_counts(a.counts, checks, s_wave, s_found).found : uniform_load(before + a.chunks);
        const bool descends = found & 1;
        if (!(found & 2)) return;
        // 4096 rows: those that begin in the part in which the first of them does, and behind the first 4096 that do
        const int64_t r0 = ((int64_t)blockIdx.x - teller) * kCompactRows, at0 = clamped(a, r0);
        // (the end of the arrays belongs to the last chunk's last part)
        const int64_t chunk = min(at0 / a.chunk, (int64_t)a.chunks - 1), c0 = chunk * a.chunk, c1 = min(c0 + a.chunk, a.nnz);
        const int64_t parts = max((c1 - c0 + kCompactPart - 1) / kCompactPart, (int64_t)1);
        const int64_t part = min((at0 - c0) / kCompactPart, parts - 1), begin = c0 + part * kCompactPart;
        const int64_t end = min(begin + kCompactPart, c1);
        const bool rest = chunk == a.chunks - 1 && part == parts - 1;
        const int64_t from = (begin == 0 ? 0 : first_row_from(a.row_ptr, a.rows, begin)) + kCompactRows;
        if (from >= r0 + kCompactRows || descends) return;
        int64_t base = a.counts ? sum_counts(a.counts, checks + (int)chunk, s_wave, s_found).survivors : before[chunk];
        float v[16];
        unsigned long long word;
        uint32_t prefix, all;
        for (int64_t p = c0; p < begin; p += kCompactPart) {
            load_part(a.val, p, c1, v);
            drop_outside(range, p, v);
            prefix = part_words(v, s_mask, &word, &all);
            base += all;
            __syncthreads();
        }
        load_part(a.val, begin, c1, v);
        drop_outside(range, begin, v);
        prefix = part_words(v, s_mask, &word, &all);
#pragma unroll 4
        for (int u = 0; u < kCompactRows / kCompactThreads; ++u) {
            const int64_t r = r0 + u * kCompactThreads + threadIdx.x;
            const int64_t at = r <= a.rows ? clamped(a, r) : INT64_MAX;
            const bool here = r >= from && r <= a.rows && (at < end || rest);
            const int n = survivors_before(here ? (int)(at - begin) : 0, word, prefix);
            if (here) new_row_ptr[r] = base + n;
        }
        return;
    }
    const int64_t c0 = (int64_t)b * a.chunk, c1 = min(c0 + a.chunk, a.nnz);
    const bool last_chunk = b == a.chunks - 1;
    // (before the part is requested: beside it, the registers of the sums cost a wave per SIMD)
    int64_t base;
    bool descends;
    if (a.counts) {
        const CountSum sum = sum_counts(a.counts, checks + b, s_wave, s_found);
        base = sum.survivors;
        descends = sum.found & 1;
    } else {
        base = before[b];
        descends = uniform_load(before + a.chunks) & 1;
    }
    int64_t row = c0 == 0 ? 0 : first_row_from(a.row_ptr, a.rows, c0);
    for (int64_t begin = c0; begin < c1 || begin == c0; begin += kCompactPart) {
        const int64_t end = min(begin + kCompactPart, c1);
        float v[16];
        int32_t c[16];
        load_part(a.val, begin, c1, v);
        load_part(a.col, begin, c1, c);
        drop_outside(range, begin, v);
        unsigned long long word;
        uint32_t all;
        const uint32_t prefix = part_words(v, s_mask, &word, &all);
        if (descends) return;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int w = u * (kCompactThreads / 64) + wave;
            const unsigned long long m = __ballot(survives(v[u]));
            const int first = __builtin_amdgcn_readlane((int)prefix, __builtin_amdgcn_readfirstlane(w));
            const int64_t p = base + first + __popcll(m & ((1ull << lane) - 1ull));
            if (survives(v[u]) && p < a.capacity) {
                out_col[p] = c[u];
                out_val[p] = v[u];
            }
        }
        // the rows that begin in this part, the first 4096 of them; behind the last part all that are left, row_ptr's end
        // among them
        const bool rest = last_chunk && end >= c1;
        for (int64_t r0 = row; r0 < row + kCompactRows; r0 += kCompactThreads) {
            const int64_t r = r0 + threadIdx.x;
            const int64_t at = r <= a.rows ? min(max((int64_t)a.row_ptr[r], begin), rest ? end : INT64_MAX) : INT64_MAX;
            const bool here = r <= a.rows && (at < end || rest);
            const int n = survivors_before(here ? (int)(at - begin) : 0, word, prefix);
            if (here) new_row_ptr[r] = base + n;
            if (!__syncthreads_and(here)) break;
        }
        base += all;
        if (end >= c1) break;
        row = first_row_from(a.row_ptr, a.rows, end);
        __syncthreads();
    }
}

// ---- row pointers that go down somewhere --------------------------------------------------------
// The largest of the row pointers up to each, by one block.
template <typename RP>
__global__ __launch_bounds__(1024) void k_compact_ascending(CompactArgs<RP> a, int64_t *__restrict__ ascending) {
    __shared__ int64_t s_most[1024];
    int64_t carry = 0;
    for (int64_t r0 = 0; r0 <= a.rows; r0 += 1024) {
        const int64_t r = r0 + threadIdx.x;
        int64_t x = r <= a.rows ? max(clamped(a, r), carry) : carry;
        s_most[threadIdx.x] = x;
        __syncthreads();
        for (unsigned d = 1; d < 1024; d <<= 1) {
            const int64_t left = threadIdx.x >= d ? s_most[threadIdx.x - d] : 0;
            __syncthreads();
            x = max(x, left);
            s_most[threadIdx.x] = x;
            __syncthreads();
        }
        if (r <= a.rows) ascending[r] = x;
        carry = s_most[1023];
        __syncthreads();
    }
}
// The new row pointers in their place, a wave per row: the survivors of the chunk before the row's first entry.
__global__ __launch_bounds__(256) void k_compact_row_ptr(int64_t *__restrict__ row_ptr, int64_t rows, const float *__restrict__ val,
                                                         int64_t chunk, int chunks, const int64_t *__restrict__ before) {
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r > rows) return;
    const int64_t at = row_ptr[r], b = min(at / chunk, (int64_t)chunks - 1);
    uint32_t n = 0;
    for (int64_t e = max(b * chunk, before[chunks + 1]) + lane_id(); e < at; e += 64) n += survives(val[e]) ? 1u : 0u;
    n = wave_sum(n);
    if (lane_id() == 0) row_ptr[r] = before[b] + n;
}

template <typename RP>
static CompactArgs<RP> compact_args(const tsp_csr *C) {
    return {static_cast<const RP *>(C->row_ptr), C->col_idx, static_cast<const float *>(C->val), C->rows, C->nnz, C->rows,
            compact_chunk(C->nnz), (int)compact_chunks(C->nnz), nullptr, C->nnz};
}
// Blocks of the counting pass; whether those of the copying pass add up their counts
template <typename RP>
static int64_t count_blocks(const CompactArgs<RP> &a) { return a.row_blocks(kCheckRows) + a.chunks; }
template <typename RP>
static bool sums_in_copy(const CompactArgs<RP> &a) { return count_blocks(a) <= kCompactSums; }
template <typename RP>
static dim3 compact_grid(const CompactArgs<RP> &a, int rows_per_block) {
    return dim3((unsigned)(a.chunks + a.row_blocks(rows_per_block)));
}
template <typename RP>
static void compact_copy(tsp_context *ctx, const CompactArgs<RP> &a, const int64_t *before, int64_t *row_ptr, int32_t *col, float *val, bool tell,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_compact_fill<RP>, dim3((unsigned)((a.counts ? 1 : 0) + a.row_blocks(kCompactRows) + a.chunks)), dim3(kCompactThreads), 0, s, a,
                       before, row_ptr, col, val, ctx->d_scalars, ctx->h_scalars_dev, tell ? ++ctx->publish_tag : (int64_t)0);
}
// The counts, and where no copying pass behind them does it, the sums and the total to the host
template <typename RP>
static void compact_launch(tsp_context *ctx, const CompactArgs<RP> &a, uint32_t *count, int64_t *before, bool copy_tells, hipStream_t s) {
    hipLaunchKernelGGL(k_compact_count<RP>, compact_grid(a, kCheckRows), dim3(kCompactThreads), 0, s, a, count, before, ctx->d_scalars);
    if (a.counts && copy_tells) return;
    if (a.counts) hipLaunchKernelGGL(k_compact_fill<RP>, dim3(1), dim3(kCompactThreads), 0, s, a, before, (int64_t *)nullptr, (int32_t *)nullptr,
                                     (float *)nullptr, ctx->d_scalars, ctx->h_scalars_dev, ++ctx->publish_tag);
    else hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(1024), 0, s, count, a.chunks, before, ctx->d_scalars, ctx->h_scalars_dev,
                       ++ctx->publish_tag);
}
// The pass again for a matrix whose row pointers go down, with ascending ones in `row_ptr`: the counts, for which it waits.
template <typename RP>
static int compact_descending(tsp_context *ctx, const CompactArgs<RP> &a, int64_t *row_ptr, uint32_t *count, int64_t *before,
                              CompactArgs<int64_t> *again, hipStream_t s) {
    hipLaunchKernelGGL(k_compact_ascending<RP>, dim3(1), dim3(1024), 0, s, a, row_ptr);
    *again = {row_ptr, a.col, a.val, -1, a.nnz, a.rows, a.chunk, a.chunks, nullptr, a.nnz};
    compact_launch(ctx, *again, count, before, false, s);
    TSP_HIP_CHECK(ctx, hipGetLastError());
    return wait_published_scalars(ctx, ctx->publish_tag, s);
}
static void compact_descending_fill(tsp_context *ctx, const CompactArgs<int64_t> &a, const int64_t *before, int64_t *row_ptr, int32_t *col, float *val, hipStream_t s) {
    compact_copy(ctx, a, before, row_ptr, col, val, false, s);
    hipLaunchKernelGGL(k_compact_row_ptr, dim3((unsigned)((a.last + 4) / 4)), dim3(256), 0, s, row_ptr, a.last, a.val, a.chunk,
                       a.chunks, before);
}

template <typename RP>
static int compact_run(tsp_context *ctx, const tsp_csr *C, tsp_csr *out, hipStream_t s, bool *taken) {
    CompactArgs<RP> a = compact_args<RP>(C);
    uint32_t *count = ctx_alloc_n<uint32_t>(ctx, (size_t)count_blocks(a) + 3, s);      // (read four at a time)
    int64_t *before = ctx_alloc_n<int64_t>(ctx, (size_t)a.chunks + 3, s);
    int64_t *new_row_ptr = nullptr;
    int32_t *col = nullptr;
    float *val = nullptr;
    auto fail = [&](int code) {
        ctx_free(ctx, count, s);
        ctx_free(ctx, before, s);
        ctx_free(ctx, new_row_ptr, s);
        ctx_free(ctx, col, s);
        ctx_free(ctx, val, s);
        return code;
    };
    if (!count || !before) return fail(TSP_ERR_ALLOC_FAILED);
    if (sums_in_copy(a)) a.counts = reinterpret_cast<const uint16_t *>(count);
    // Without waiting for the new nnz, into arrays for as many entries as the last matrix of these sizes had left and some more, where it
    // was to be copied (3 us saved, of 52; a copy in vain where this one has more left); for a caller that takes C as it is where nothing is dropped the blocks of the copy look at that first
    if (taken && a.counts) a.mark = ctx->publish_tag + 1;
    CompactHint &hint = ctx->compact_hints.find({{C->rows, C->nnz, C->cols, 0, 0, 0}}, [](CompactHint &) {});
    const int64_t expected = std::min(hint.nnz + hint.nnz / 16, C->nnz);
    bool ahead = a.counts && hint.nnz >= 0 && !(taken && hint.nnz == C->nnz) && hint.ahead.allowed();
    auto allocate_result = [&](int64_t entries) {
        if (!new_row_ptr) new_row_ptr = ctx_alloc_n<int64_t>(ctx, (size_t)C->rows + 1, s);
        col = ctx_alloc_n<int32_t>(ctx, (size_t)entries, s);
        val = ctx_alloc_n<float>(ctx, (size_t)entries, s);
        return new_row_ptr && col && val;
    };
    auto drop_result = [&]() {
        for (auto p : {(void **)&new_row_ptr, (void **)&col, (void **)&val}) {
            ctx_free(ctx, *p, s);
            *p = nullptr;
        }
        ahead = false;
    };
    if (ahead && !allocate_result(expected)) drop_result();
    compact_launch(ctx, a, count, before, ahead, s);
    if (ahead) {
        CompactArgs<RP> bounded = a;
        bounded.capacity = expected;
        compact_copy(ctx, bounded, before, new_row_ptr, col, val, true, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(hip_fail(ctx, e));
    int rc = wait_published_scalars(ctx, ctx->publish_tag, s);            // host synchronisation: the new nnz
    if (rc) return fail(rc);
    const bool descends = ctx->h_scalars[S_DESCENDS] != 0;
    hint.nnz = ctx->h_scalars[S_C_NNZ];
    const bool fits = !descends && hint.nnz <= expected && !(taken && hint.nnz == C->nnz);
    if (!ahead) hint.ahead.other_way(fits);
    else if (fits) hint.ahead.taken();
    else hint.ahead.missed();
    if (ahead && !fits) drop_result();
    CompactArgs<int64_t> again{};
    if (descends) {
        new_row_ptr = ctx_alloc_n<int64_t>(ctx, (size_t)C->rows + 1, s);
        rc = new_row_ptr ? compact_descending(ctx, a, new_row_ptr, count, before, &again, s) : (int)TSP_ERR_ALLOC_FAILED;
        if (rc) return fail(rc);
    }
    const int64_t nnz = ctx->h_scalars[S_C_NNZ];
    if (taken && !descends && nnz == C->nnz) {                        // nothing to drop: the caller's arrays are the result
        fail(TSP_OK);                                    // (releases the scratch arrays)
        *out = *C;
        *taken = true;
        return TSP_OK;
    }
    if (!ahead) {
        if (!allocate_result(nnz)) return fail(TSP_ERR_ALLOC_FAILED);
        if (descends) compact_descending_fill(ctx, again, before, new_row_ptr, col, val, s);
        else compact_copy(ctx, a, before, new_row_ptr, col, val, false, s);
        e = hipGetLastError();
        if (e != hipSuccess) return fail(hip_fail(ctx, e));
    }
    ctx_free(ctx, count, s);
    ctx_free(ctx, before, s);
    out->rows = C->rows;
    out->cols = C->cols;
    out->nnz = nnz;
    out->row_ptr = new_row_ptr;
    out->col_idx = col;
    out->val = val;
    out->row_ptr_type = TSP_I64;
    out->val_type = TSP_F32;
    return TSP_OK;
}

int compact_zeros(tsp_context *ctx, const tsp_csr *C, tsp_csr *out, hipStream_t s, bool *taken) {
    std::memset(out, 0, sizeof(*out));
    if (taken) *taken = false;
    if (C->rows < 0 || C->cols < 0 || C->nnz < 0 || !C->row_ptr) return TSP_ERR_INVALID_ARG;
    if (C->val_type != TSP_F32) return TSP_ERR_INVALID_ARG;
    if (C->nnz > 0 && (!C->col_idx || !C->val)) return TSP_ERR_INVALID_ARG;
    if (C->rows >= INT32_MAX - 16) return TSP_ERR_INDEX_OVERFLOW;
    if (C->row_ptr_type == TSP_I64) return compact_run<int64_t>(ctx, C, out, s, taken);
    if (C->row_ptr_type == TSP_I32) return compact_run<int32_t>(ctx, C, out, s, taken);
    return TSP_ERR_INVALID_ARG;
}

// ---- the same compaction without any allocation (tsp_compact_zeros_static) -----------------------
// The counts and the prefix sums of the chunks, which compact_run takes from the handle's allocator, live in a file-scope
// device array instead.  Every device the library runs on holds its own
// copy of the array, at its own address, until the process ends; the address is looked up once per device
// (static_scratch_setup) and only that pointer is ever handed to kernels.
constexpr int64_t kStaticMaxRows = TSP_COMPACT_STATIC_MAX_ROWS;
constexpr size_t kStaticCountBytes = (size_t)kCompactChunks * sizeof(uint32_t);
constexpr size_t kStaticBeforeBytes = (size_t)(kCompactChunks + 32) * sizeof(int64_t);
static __device__ __align__(256) unsigned char scratch[kStaticBeforeBytes + kStaticCountBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static unsigned char *g_scratch_ptr[kMaxDevices];      // device address of `scratch` on every device seen so far

// Device address of the scratch array on the current device (looked up on the first call per device).
int static_scratch_setup(tsp_context *ctx, unsigned char **ptr) {
    int device = -1;
    TSP_HIP_CHECK(ctx, hipGetDevice(&device));
    if (device < 0 || device >= kMaxDevices) return TSP_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        TSP_HIP_CHECK(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return hip_fail(ctx, hipErrorInvalidSymbol);
        g_scratch_ptr[device] = static_cast<unsigned char *>(p);
    }
    if (ptr) *ptr = g_scratch_ptr[device];
    return TSP_OK;
}

template <typename RP>
static int compact_run_static(tsp_context *ctx, const tsp_csr *C, tsp_csr *out, hipStream_t s) {
    unsigned char *base = nullptr;
    int rc = static_scratch_setup(ctx, &base);
    if (rc) return rc;
    int64_t *before = reinterpret_cast<int64_t *>(base);
    uint32_t *count = reinterpret_cast<uint32_t *>(base + kStaticBeforeBytes);
    CompactArgs<RP> a = compact_args<RP>(C);
    if (sums_in_copy(a)) a.counts = reinterpret_cast<const uint16_t *>(count);
    int64_t *const new_row_ptr = static_cast<int64_t *>(out->row_ptr);
    float *const val = static_cast<float *>(out->val);
    // (nothing in the scratch array has to start at zero; the copy does not wait for the host)
    compact_launch(ctx, a, count, before, true, s);
    compact_copy(ctx, a, before, new_row_ptr, out->col_idx, val, a.counts != nullptr, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e);
    rc = wait_published_scalars(ctx, ctx->publish_tag, s);       // host synchronisation: the new nnz
    if (rc) return rc;
    if (ctx->h_scalars[S_DESCENDS]) {
        CompactArgs<int64_t> again{};
        rc = compact_descending(ctx, a, new_row_ptr, count, before, &again, s);
        if (rc) return rc;
        compact_descending_fill(ctx, again, before, new_row_ptr, out->col_idx, val, s);
        TSP_HIP_CHECK(ctx, hipGetLastError());
    }
    const int64_t nnz = ctx->h_scalars[S_C_NNZ];
    out->rows = C->rows;
    out->cols = C->cols;
    out->nnz = nnz;
    out->row_ptr_type = TSP_I64;
    out->val_type = TSP_F32;
    return TSP_OK;
}

}  // namespace tsp

using namespace tsp;

extern "C" int tsp_compact_zeros_static(tsp_handle ctx, const tsp_csr *C, tsp_csr *out, void *stream) {
    if (!ctx || !C || !out || C == out) return TSP_ERR_INVALID_ARG;
    if (C->rows < 0 || C->cols < 0 || C->nnz < 0 || !C->row_ptr || !out->row_ptr) return TSP_ERR_INVALID_ARG;
    if (C->val_type != TSP_F32) return TSP_ERR_INVALID_ARG;
    if (C->nnz > 0 && (!C->col_idx || !C->val || !out->col_idx || !out->val)) return TSP_ERR_INVALID_ARG;
    if (C->rows < 1 || C->rows > kStaticMaxRows) return TSP_ERR_UNSUPPORTED;      // the scratch array has a fixed size
    hipStream_t s = (hipStream_t)stream;
    if (C->row_ptr_type == TSP_I64) return compact_run_static<int64_t>(ctx, C, out, s);
    if (C->row_ptr_type == TSP_I32) return compact_run_static<int32_t>(ctx, C, out, s);
    return TSP_ERR_INVALID_ARG;
}

extern "C" int tsp_compact_zeros(tsp_handle ctx, const tsp_csr *C, tsp_csr *out, void *stream) {
    if (!ctx || !C || !out || C == out) return TSP_ERR_INVALID_ARG;
    return compact_zeros(ctx, C, out, (hipStream_t)stream, nullptr);
}
