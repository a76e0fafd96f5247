// Conversion kernels: CSR or dense device matrix -> GCOO arrays (Section 3.1, Algorithm 1).
//
// All kernels are deterministic: the slot of every entry is computed from counts and
// wave-wide ballots, never from the arrival order of atomics, so the arrays come out
// bit-identical from run to run (and equal to the definition: per group, ordered by
// column, then row, then input position).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace gcoo {

constexpr int kWave = 64;

// What the host wants to know about a CSR input before it sizes anything: out[0] = nnz = row_ptr[m],
// out[1] = entries of the largest group.  The work of one workgroup of THREADS threads.
template <int THREADS>
__device__ __forceinline__ void group_stats_block(const int32_t* __restrict__ row_ptr, int64_t m, int32_t p, int64_t g,
                                                  unsigned long long* __restrict__ out)
{
    __shared__ int32_t part[THREADS / 64];
    int32_t mx = 0;
    for (int64_t q = threadIdx.x; q < g; q += THREADS) {
        const int64_t r0 = q * p, r1 = (r0 + p < m) ? r0 + p : m;
        const int32_t n = row_ptr[r1] - row_ptr[r0];
        mx = n > mx ? n : mx;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int32_t o = __shfl_down(mx, d, kWave);
        mx = o > mx ? o : mx;
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < THREADS / 64; ++i) mx = part[i] > mx ? part[i] : mx;
        const int32_t last = row_ptr[m];
        out[0] = last < 0 ? ~0ull : (unsigned long long)last;
        out[1] = (unsigned long long)mx;
    }
}

// A kernel's answer to the host, straight to pinned host memory.
__device__ __forceinline__ void tell_host(unsigned long long* host, unsigned long long a)
{
    __hip_atomic_store(host, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// nnz = row_ptr[m] of a CSR input on the device.  One thread.
__global__ void read_entry_count(const int32_t* __restrict__ row_ptr, int64_t m, unsigned long long* __restrict__ host)
{
    const int32_t last = row_ptr[m];
    tell_host(host, last < 0 ? 1ull << 62 : (unsigned long long)last);
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1, step 1 for a CSR input.  CSR is row-major, so the entries of group q are the
// contiguous CSR range [row_ptr[q*p], row_ptr[min((q+1)*p, m)]): the count and the prefix sum
// are two reads of row_ptr.  One thread per group; thread g also writes the sentinel.
// 256 threads per workgroup, ceil((g+1)/256) workgroups (ceil((m+1)/256) with `row_start` given, which receives the
// clamped offsets of all rows); with `stats` given, one workgroup more, which computes the statistics above in the same launch.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void group_index_from_row_ptr(const int32_t* __restrict__ row_ptr, int64_t m, int32_t p, int64_t g,
                                                                 int32_t nnz, int32_t* __restrict__ gIdxes,
                                                                 int32_t* __restrict__ nnzPerGroup, unsigned long long* __restrict__ stats,
                                                                 uint32_t* __restrict__ bad_col, int32_t* __restrict__ row_start)
{
    if (stats && blockIdx.x == gridDim.x - 1) {                   // the whole workgroup
        // bad_col[0] is set by the sort that follows if it meets a column out of range, bad_col[1] counts the rows it lists as long,
        // bad_col[2] is set for uneven rows, bad_col[3] counts the longest ones
        if (threadIdx.x < 4) bad_col[threadIdx.x] = 0u;
        group_stats_block<256>(row_ptr, m, p, g, stats);
        return;
    }
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // Offsets are clamped to [0, nnz]: with a device input whose row_ptr does not match the nnz
    // the buffer was laid out for, every later kernel still stays inside the arrays.
    auto at = [&](int64_t r) { const int32_t v = row_ptr[r]; return v < 0 ? 0 : (v > nnz ? nnz : v); };
    if (row_start && q <= m) row_start[q] = at(q);
    if (q > g) return;
    int64_t r0 = q * p;
    if (r0 > m) r0 = m;
    const int32_t b = at(r0);
    gIdxes[q] = b;
    if (q < g) {
        int64_t r1 = r0 + p;
        if (r1 > m) r1 = m;
        const int32_t n = at(r1) - b;
        nnzPerGroup[q] = n < 0 ? 0 : n;
    }
}

__device__ __forceinline__ uint64_t lanemask_lt()
{
    return (1ull << (threadIdx.x & 63)) - 1ull;   // one wave per workgroup in the kernels below
}

// Inclusive prefix sum over every stretch of LANES (16, 32 or 64) lanes of a whole wave.
template <int LANES>
__device__ __forceinline__ int32_t lanes_scan(int32_t x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    if constexpr (LANES >= 32) x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast:15, into rows 1 and 3
    if constexpr (LANES == 64) x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // row_bcast:31, into rows 2 and 3
    return x;
}

// Exclusive prefix sum over a workgroup of WAVES whole waves, 16 at the most; the total in *all.  One barrier; `sums` is free again behind the next one.
template <int WAVES>
__device__ __forceinline__ int32_t block_scan(int32_t x, int32_t* sums, int32_t* all)
{
    static_assert(WAVES <= 16, "");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t incl = lanes_scan<64>(x);
    if (lane == 63) sums[wave] = incl;
    __syncthreads();
    const int32_t waves = lanes_scan<16>(lane < WAVES ? sums[lane] : 0);
    *all = __builtin_amdgcn_readlane(waves, WAVES - 1);
    return incl - x + (wave > 0 ? __builtin_amdgcn_readlane(waves, wave - 1) : 0);
}

// Whether x holds in any thread of it.  One barrier, where __syncthreads_or() has more; `any` as `sums` above.
template <int WAVES>
__device__ __forceinline__ bool block_any(bool x, int32_t* any)
{
    const int lane = threadIdx.x & 63;
    const bool mine = __any(x);
    if (lane == 0) any[threadIdx.x >> 6] = mine;
    __syncthreads();
    return __any(lane < WAVES && any[lane] != 0);
}

// Lanes of the wave whose 8-bit digit equals this lane's, among the lanes in `active`.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool is_active)
{
    uint64_t mask = __ballot(is_active);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        bool bit = (d >> b) & 1u;
        uint64_t bb = __ballot(is_active && bit);
        mask &= bit ? bb : ~bb;
    }
    return mask;
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1, step 2 for a CSR input: one pass of a stable least-significant-digit radix sort
// of every group's entries on an 8-bit digit of the column index.  One workgroup of kSortWaves
// waves per group.
//
// The CSR order of a group's entries is (row, input position); sorting that stably by column
// gives (column, row, input position).  Each pass is a counting sort.  The group's entries are
// cut into kSortWaves contiguous parts, one per wave.  Every wave counts the digits of its part
// (LDS, a histogram of its own); from those counts each (wave, digit) gets the slot where the
// wave's first entry with that digit goes: digit base + what earlier waves hold of the digit.
// Then every wave walks its part 64 entries at a time, in order, and gives each entry
// slot = that running base + number of earlier entries of the 64 with the same digit (ballots).
// Nothing depends on timing: counts are sums, ranks come from ballots.
//
// FIRST: the source is the CSR input itself (row of an entry = search in row_ptr; columns are forced
// into [0, kcols) and *bad_col is set if one was outside); otherwise the source is the (cols, rows,
// values) triple written by the previous pass.
//
// BY_ROW: the finished arrays are the source, the digit is the row inside the group: the entries come out in (row,
// column) order, which is what the row-by-row kernel reads when the input was no CSR matrix.
//
// nb > 0: the workgroup sorts one bucket of one group instead of a whole group.  The pass before
// it has sorted the group by the digit above (col >> 8, nb values); bucket b of group q is the
// stretch of the group with that digit equal to b, found by two binary searches, and it is sorted
// in place (inside its own stretch of the destination) by the low digit.  High digit first keeps
// the stores of both passes close together: consecutive entries of a CSR row fall into the same
// bucket in the first pass, and a bucket's stretch is a few kilobytes in the second, where the
// low digit first scatters every store of both passes over the whole group.
// ---------------------------------------------------------------------------------------------
constexpr int kSortWaves = 16;          // waves of the workgroup that sorts a whole group
constexpr int kSortBucketWaves = 4;     // and of the one that sorts one bucket of a group (about a thousand entries)

enum SortPass { kSortFirst, kSortNext, kSortByRow };

// What the row-by-row kernel reads, as far as the sorts write it (nothing where `cols` is null).
struct RowsOut {
    int32_t* cols;             // the entries in row order
    float* vals;
    int32_t* start;            // where the rows begin (read by kSortFirst, written by kSortByRow)
    int32_t* long_rows;        // long_room places for the rows of more than `long_row` entries: the longest from the front, long_count[2] of them, the others from the back, long_count[0]
    int32_t* long_count;
    int32_t long_row, long_room;
};
// The longest rows are taken first, so that a product does not end with one of them (power-law rows, product alone, over 91 matrices of 4200 to 20000 rows, N = 257 to 900: 3.4 % less than with
// all of them in one list; N = 40 to 256 level).
constexpr int kRowsLongFront = 3;
__device__ __forceinline__ void list_long_row(const RowsOut& out, int32_t row, int32_t entries)
{
    if (entries <= out.long_row) return;
    const bool front = entries > kRowsLongFront * (int64_t)out.long_row;
    const int32_t at = atomicAdd(out.long_count + (front ? 2 : 0), 1);
    if (at < out.long_room) out.long_rows[front ? at : out.long_room - 1 - at] = row;
}

template <SortPass PASS, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void sort_groups_by_col_digit(
    const int32_t* __restrict__ gIdxes, const int32_t* __restrict__ row_ptr, int64_t m, int32_t p,
    const int32_t* __restrict__ src_cols, const int32_t* __restrict__ src_rows, const float* __restrict__ src_vals,
    int32_t* __restrict__ dst_cols, int32_t* __restrict__ dst_rows, float* __restrict__ dst_vals, int shift, int32_t nb,
    int32_t kcols, uint32_t* __restrict__ bad_col, RowsOut out)
{
    constexpr bool FIRST = PASS == kSortFirst, BY_ROW = PASS == kSortByRow;
    // FIRST: a column of the input outside [0, kcols) is stored clamped into that range and reported in
    // *bad_col, so that no later kernel forms an address outside B from it
    const int64_t q = nb > 0 ? blockIdx.x / nb : blockIdx.x;
    const int32_t row_first = (int32_t)(q * p);
    auto in_range = [&](int32_t c) { return FIRST ? (c < 0 ? 0 : (c >= kcols ? kcols - 1 : c)) : c; };
    // the digit of an entry: 8 bits of its column, or (BY_ROW) its row inside the group
    auto digit = [&](int32_t x) { return BY_ROW ? (uint32_t)(x - row_first) : ((uint32_t)in_range(x) >> shift) & 255u; };
    __shared__ int32_t slot_of[WAVES][256];      // counts, then running slots, per wave and digit
    __shared__ int32_t total[256];
    __shared__ int32_t rp_s[FIRST ? 257 : 1];         // FIRST: row_ptr of the group's rows (at most 256 + 1), searched per entry
    __shared__ int32_t range_s[2];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t beg = gIdxes[q], end = gIdxes[q + 1];
    if (beg >= end && !BY_ROW) return;
    if (nb > 0) {
        // threads 0 and 1: first entry of the group whose high digit is >= b, and >= b + 1
        if (tid < 2) {
            const int32_t want = (int32_t)(blockIdx.x - q * nb) + tid;
            int32_t lo = beg, hi = end;
            while (lo < hi) {
                const int32_t mid = lo + (hi - lo) / 2;
                if ((src_cols[mid] >> 8) < want) lo = mid + 1; else hi = mid;
            }
            range_s[tid] = lo;
        }
        __syncthreads();
        beg = range_s[0];
        end = range_s[1];
        if (beg >= end) return;                      // the whole workgroup
    }
    if (FIRST) {
        const int64_t r_lo = q * p;
        const int64_t r_hi = (r_lo + p < m) ? r_lo + p : m;
        static_assert(!FIRST || WAVES * kWave >= 257, "one thread per row of the group, and one more");
        if (tid <= r_hi - r_lo) rp_s[tid] = row_ptr[r_lo + tid];     // the barriers below publish it
        if (out.cols && tid < r_hi - r_lo) list_long_row(out, (int32_t)r_lo + tid, out.start[r_lo + tid + 1] - out.start[r_lo + tid]);
    }
    // part of wave wv: whole 64-entry tiles
    const int32_t tiles = (end - beg + kWave - 1) / kWave;
    const int32_t tiles_per = (tiles + WAVES - 1) / WAVES;
    const int32_t pb = beg + wv * tiles_per * kWave;
    const int32_t pe = (pb + tiles_per * kWave < end) ? pb + tiles_per * kWave : end;

    for (int i = tid; i < WAVES * 256; i += WAVES * kWave) (&slot_of[0][0])[i] = 0;
    __syncthreads();
    // (four loads in flight per lane: a wave's part is some thirty tiles, and one load at a time made the pass a chain
    // of memory latencies)
    for (int32_t e = pb + lane; e < pe; e += 4 * kWave) {
        int32_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = e + u * kWave < pe ? (BY_ROW ? src_rows : src_cols)[e + u * kWave] : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (e + u * kWave < pe) atomicAdd(&slot_of[wv][digit(c[u])], 1);   // counts only: order-free
    }
    __syncthreads();
    if (tid < 256) {
        int32_t run = 0;
        for (int w = 0; w < WAVES; ++w) {
            const int32_t c = slot_of[w][tid];
            slot_of[w][tid] = run;
            run += c;
        }
        total[tid] = run;
    }
    __syncthreads();
    if (wv == 0) {
        // exclusive scan of the 256 digit totals: lane owns digits 4*lane .. 4*lane+3
        const int32_t c0 = total[4 * lane], c1 = total[4 * lane + 1], c2 = total[4 * lane + 2], c3 = total[4 * lane + 3];
        const int32_t sum = c0 + c1 + c2 + c3;
        int32_t incl = sum;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t t = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += t;
        }
        const int32_t ex = incl - sum;
        total[4 * lane] = ex;
        total[4 * lane + 1] = ex + c0;
        total[4 * lane + 2] = ex + c0 + c1;
        total[4 * lane + 3] = ex + c0 + c1 + c2;
    }
    __syncthreads();
    for (int i = tid; i < WAVES * 256; i += WAVES * kWave) (&slot_of[0][0])[i] += total[i & 255];
    if (BY_ROW) {                                    // where the rows of the group begin; the last group adds the end
        if (tid < p && row_first + tid < m) {
            out.start[row_first + tid] = beg + total[tid];
            list_long_row(out, row_first + tid, total[tid + 1] - total[tid]);
        }
        if (tid == 0 && row_first + p >= m) out.start[m] = end;
    }
    __syncthreads();

    // From here on the waves do not meet again: a wave's LDS operations execute in order, and the
    // volatile accesses keep the compiler from reordering the read of a slot and its update.
    volatile int32_t* my_slot = slot_of[wv];
    const int64_t r_lo = q * p;
    const int64_t r_hi = (r_lo + p < m) ? r_lo + p : m;
    const uint64_t lt = lanemask_lt();
    // the loads of the next tile are issued before this tile is ranked and stored
    int32_t col_next = 0, row_next = 0;
    float val_next = 0.0f;
    auto request = [&](int32_t t) {
        const int32_t e = t + lane;
        if (e < pe) {
            col_next = src_cols[e];
            val_next = src_vals[e];
            if (!FIRST) row_next = src_rows[e];
        }
    };
    request(pb);
    for (int32_t t0 = pb; t0 < pe; t0 += kWave) {
        const int32_t e = t0 + lane;
        const bool act = e < pe;
        int32_t col = col_next, row = row_next;
        float val = val_next;
        if (t0 + kWave < pe) request(t0 + kWave);
        if (act) {
            if (FIRST) {
                const int32_t c = in_range(col);
                if (c != col) { *bad_col = 1u; col = c; }
                if (out.cols) {                                   // the entries in row order, as they came
                    out.cols[e] = col;
                    out.vals[e] = val;
                }
                // row r with row_ptr[r] <= e < row_ptr[r+1]; empty rows are skipped by the upper bound
                int32_t lo = 0, hi = (int32_t)(r_hi - r_lo);      // answer in [lo, hi), relative to the group's first row
                while (hi - lo > 1) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (rp_s[mid] <= e) lo = mid; else hi = mid;
                }
                row = (int32_t)r_lo + lo;
            }
        }
        const uint32_t d = BY_ROW ? (uint32_t)(row - row_first) : ((uint32_t)col >> shift) & 255u;
        const uint64_t same = match_digit(d, act);
        const int32_t before = __popcll(same & lt);
        int32_t slot = 0;
        if (act) slot = my_slot[d];
        __builtin_amdgcn_wave_barrier();
        if (act && before == 0) my_slot[d] = slot + __popcll(same);   // first lane of each digit advances it
        __builtin_amdgcn_wave_barrier();
        if (act) {
            const int32_t at = beg + slot + before;
            dst_cols[at] = col;
            if (!BY_ROW) dst_rows[at] = row;
            dst_vals[at] = val;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1 for a dense input.  The band of group q (pb rows x k columns) is cut into blocks of
// kDenseThreads*VW columns; workgroup (block, q) gives every thread VW adjacent columns, and the
// threads of a wave read 64*VW adjacent floats of a row at a time (coalesced), row after row.
//
// Step 1 (count_dense_blocks): entries != 0 per block; the last workgroup to end turns the counts into the first slot of
// every block (exclusive prefix sum, groups and blocks in order), gIdxes and nnzPerGroup.
// Bound: reading A once.  The workgroups meet only at the end of each (an atomic per wave on one address took 105 us for 4000 x 4000; see arrive()
// for one per workgroup).  With the scan behind it: 14.6 us, 15.1 with the masks.
// ---------------------------------------------------------------------------------------------
constexpr int kDenseThreads = 256;
constexpr int kDenseWorkgroups = 1024;       // of a counting launch, at most

// The words in which the workgroups of a counting launch count themselves, all zero before and after.  Arrivals at one word follow one another at
// 14 ns each, whatever XCD they come from, so workgroup i arrives at word i % words, and the last one there at the word behind them; the words are
// kTicketStride apart, since it is the line that serialises.
constexpr int kTicketWords = 32;
constexpr int kTicketStride = 16;            // 128 bytes
struct DenseTicket {
    unsigned long long* at;
    int32_t words;                           // 1 .. kTicketWords; 1: the word itself, and none behind it
};

// A word that the workgroups of one launch hand to each other across an arrival.  It has no plain access: it is stored and loaded with agent scope, that is
// past the L2 of an XCD, which is what arrive() stands on.  settled() is the ordinary load of it, for later launches.
template <typename T>
class Handed {
public:
    __device__ __forceinline__ void store(T x) { __hip_atomic_store(&word_, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ T load() const { return __hip_atomic_load(&word_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ T settled() const { return word_; }

private:
    T word_;
};

// All earlier memory operations of this wave have been done: loads are back, and what was stored with agent scope is where every XCD reads it.
__device__ __forceinline__ void wait_for_memory()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// One thread of each workgroup: true in the one that arrives last, which gets the sum of `n` over all (below 2^48).  The Handed words that this thread stored
// before it arrived are what load() reads behind the last arrival; anything else that a workgroup stores is for later launches only.
// The language's memory model knows no such order without release and acquire, which write back and invalidate the L2 of an XCD, 26 ns for each
// workgroup one after the other.  The machine's order is enough: a store with agent scope is done, for the wait in front of the arrival, when it has passed
// that L2, and a load with agent scope behind the arrival goes past it too.  The build reads the generated code for both: each arrival between
// two waits for all memory operations, nothing but masks stored in front of one without agent scope, and the last workgroup's loads with it.
// (4000 x 4000, 500 workgroups: the launch takes 25.8 us with release and acquire on one word or on 32, 17.1 with the wait on
// one word, 13.2 with the wait on 32 and 12.8 without any arrival.)
__device__ __forceinline__ bool arrive(const DenseTicket& t, unsigned long long n, unsigned long long* sum)
{
    const uint32_t all = gridDim.x, words = (uint32_t)t.words < all ? (uint32_t)t.words : all, mine = blockIdx.x % words;
    auto at_word = [&](uint32_t i, uint32_t expected) {
        unsigned long long* at = t.at + (size_t)i * kTicketStride;
        wait_for_memory();
        n += __hip_atomic_fetch_add(at, n + (1ull << 48), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + (1ull << 48);
        wait_for_memory();
        if (n >> 48 != expected) return false;
        __hip_atomic_store(at, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        n &= 0xffffffffffffull;
        return true;
    };
    if (!at_word(mine, (all - mine + words - 1) / words)) return false;
    if (t.words > 1 && !at_word((uint32_t)t.words, words)) return false;
    *sum = n;
    return true;
}

// VW adjacent floats of a row: one 16-byte load when VW = 4 (the launcher checks alignment).
template <int VW>
struct DenseVec { float x[VW]; };

template <int VW>
__device__ __forceinline__ DenseVec<VW> load_dense(const float* a)
{
    DenseVec<VW> v;
    if constexpr (VW == 4) {
        const float4 t = *reinterpret_cast<const float4*>(a);
        v.x[0] = t.x; v.x[1] = t.y; v.x[2] = t.z; v.x[3] = t.w;
    } else {
        v.x[0] = *a;
    }
    return v;
}

__device__ __forceinline__ int32_t block_sum_256(int32_t n, int32_t* part)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_down(n, d, kWave);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    return part[0] + part[1] + part[2] + part[3];
}

// Where the counts of a dense matrix live: in the buffer of the matrix, or in one of their own until nnz is known.
struct DenseCounts {
    Handed<int32_t>* blk;      // [g * nblk] first slot of a block
    int32_t* gIdxes;           // [g + 1]
    int32_t* nnzPerGroup;      // [g]
    unsigned long long* stats; // nnz, entries of the largest group
    uint64_t* masks;           // [g * k] the rows of a group that have an entry in a column, bit i for its i-th row; or null
};

// The rows among [0, nr), at most 64, in which the VW columns at `a` have an entry.  Eight loads in flight.
template <int VW>
__device__ __forceinline__ void dense_masks(const float* __restrict__ a, int64_t lda, int32_t nr, uint64_t* bits)
{
#pragma unroll
    for (int u = 0; u < VW; ++u) bits[u] = 0;
    int32_t r = 0;
    for (; r + 8 <= nr; r += 8, a += 8 * lda) {
        DenseVec<VW> v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = load_dense<VW>(a + x * lda);
#pragma unroll
        for (int u = 0; u < VW; ++u) {
            uint32_t eight = 0;
#pragma unroll
            for (int x = 0; x < 8; ++x) eight |= (v[x].x[u] != 0.0f) ? 1u << x : 0u;
            bits[u] |= (uint64_t)eight << r;
        }
    }
    for (; r < nr; ++r, a += lda) {
        const DenseVec<VW> v = load_dense<VW>(a);
#pragma unroll
        for (int u = 0; u < VW; ++u) bits[u] |= (uint64_t)(v.x[u] != 0.0f) << r;
    }
}

// Entries != 0 in rows [r0, r1), columns c .. c + VW - 1 (c < k).  Eight loads in flight.
template <int VW>
__device__ __forceinline__ int32_t count_dense_tile(const float* __restrict__ A, int64_t lda, int64_t r0, int64_t r1, int64_t c)
{
    int32_t n = 0;
    const float* a = A + r0 * lda + c;
    int64_t r = r0;
    for (; r + 8 <= r1; r += 8) {
        DenseVec<VW> v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = load_dense<VW>(a + x * lda);
        a += 8 * lda;
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int u = 0; u < VW; ++u) n += (v[x].x[u] != 0.0f) ? 1 : 0;
    }
    for (; r < r1; ++r, a += lda) {
        const DenseVec<VW> v = load_dense<VW>(a);
#pragma unroll
        for (int u = 0; u < VW; ++u) n += (v.x[u] != 0.0f) ? 1 : 0;
    }
    return n;
}

// Item i = q*nblk + b, items strided over the workgroups; thread t of block b owns columns (b*kDenseThreads + t)*VW .. +VW-1 of the
// band (k % VW == 0 when VW > 1).  `host` may be null.  MASKS: out.masks is written as well (p <= 64).
template <int VW, bool MASKS>
__global__ __launch_bounds__(kDenseThreads) void count_dense_blocks(const float* __restrict__ A, int64_t lda, int64_t m, int64_t k, int32_t p,
                                                                     int64_t nblk, int64_t g, DenseCounts out,
                                                                     DenseTicket ticket, unsigned long long* __restrict__ host)
{
    __shared__ int32_t part[4];
    __shared__ int32_t last_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t items = g * nblk;
    for (int64_t i = blockIdx.x; i < items; i += gridDim.x) {
        const int64_t q = i / nblk, b = i - q * nblk;
        const int64_t c = (b * kDenseThreads + tid) * VW;
        const int64_t r0 = q * p, r1 = (r0 + p < m) ? r0 + p : m;
        int32_t n = 0;
        if (c < k) {
            if constexpr (MASKS) {
                uint64_t bits[VW];
                dense_masks<VW>(A + r0 * lda + c, lda, (int32_t)(r1 - r0), bits);
#pragma unroll
                for (int u = 0; u < VW; ++u) n += __popcll(bits[u]);
                uint64_t* to = out.masks + q * k + c;
#pragma unroll
                for (int u = 0; u < VW; ++u) to[u] = bits[u];
            } else {
                n = count_dense_tile<VW>(A, lda, r0, r1, c);
            }
        }
        const int32_t tot = block_sum_256(n, part);
        // written where every XCD sees it, before this workgroup's arrival is counted
        if (tid == 0) out.blk[i].store(tot);
    }
    if (tid == 0) {
        unsigned long long none;
        last_s = arrive(ticket, 0, &none);
    }
    __syncthreads();
    if (!last_s) return;                                                  // the whole workgroup

    // The last workgroup: 1024 counts at a time, four per thread.
    int64_t carry = 0;
    __shared__ int64_t wsum[4];
    for (int64_t t0 = 0; t0 < items; t0 += 4 * kDenseThreads) {
        int32_t x[4];
        const int64_t i0 = t0 + 4 * tid;
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = i0 + u < items ? out.blk[i0 + u].load() : 0;
        const int64_t mine = (int64_t)x[0] + x[1] + x[2] + x[3];
        int64_t incl = mine;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int64_t t = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += t;
        }
        __syncthreads();
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        int64_t at = carry + incl - mine;
        for (int j = 0; j < w; ++j) at += wsum[j];
        carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // (a total above INT32_MAX is rejected by the host)
            if (i0 + u < items) out.blk[i0 + u].store((int32_t)(at > 0x7fffffffLL ? 0x7fffffffLL : at));
            at += x[u];
        }
    }
    __syncthreads();
    const int32_t total = (int32_t)(carry > 0x7fffffffLL ? 0x7fffffffLL : carry);
    int32_t mx = 0;
    for (int64_t q = tid; q <= g; q += kDenseThreads) {
        auto first = [&](int64_t gq) {
            return gq < g && nblk > 0 ? out.blk[gq * nblk].load() : total;
        };
        const int32_t at = first(q);
        out.gIdxes[q] = at;
        if (q < g) {
            const int32_t n = first(q + 1) - at;
            out.nnzPerGroup[q] = n;
            mx = n > mx ? n : mx;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int32_t o = __shfl_down(mx, d, kWave);
        mx = o > mx ? o : mx;
    }
    if (lane == 0) part[w] = mx;
    __syncthreads();
    if (tid == 0) {
        for (int j = 1; j < 4; ++j) mx = part[j] > mx ? part[j] : mx;
        out.stats[0] = (unsigned long long)carry;
        out.stats[1] = (unsigned long long)mx;
        if (host) {
            wait_for_memory();
            tell_host(host, (unsigned long long)carry);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1, step 2 for a dense input (fill_dense_blocks), same blocks as step 1.  Inside a
// group the entries are ordered by (column, row), so the entries of block b come right after
// those of blocks 0..b-1, column by column, and inside a column by row.  Thread c counts the
// entries of its columns, a workgroup-wide exclusive prefix sum of those counts gives the first
// slot of every column, and the thread writes each entry to its final slot.  No sort, no atomics: the slot of an entry is a
// function of the matrix alone.
// SMALL (at most 64 rows per group): a first walk leaves a bit per element behind, and only the elements that are entries
// are read a second time, the next one of each column together; taller groups walk the columns again.
// (4000 x 4000, 2 %: 32 us walking twice, 19 with the bits.)  Where the count has left the bits in memory fill_dense_masked() or fill_dense_groups() does this step.
// The launch also puts the index arrays in place where they were counted elsewhere (`from`), and clears zeroed[0..3] and, where given, the
// ticket of the count that follows.
// ---------------------------------------------------------------------------------------------
template <int THREADS = kDenseThreads>
__device__ __forceinline__ void place_dense_counts(const DenseCounts& from, const DenseCounts& to, int64_t g, uint32_t* zeroed, unsigned long long* ticket)
{
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < 4) zeroed[tid] = 0u;
    if (blockIdx.x == 0 && tid == 4 && ticket) *ticket = 0ull;
    if (from.gIdxes != to.gIdxes) {
        if (blockIdx.x == 0 && tid < 2) to.stats[tid] = from.stats[tid];
        for (int64_t q = (int64_t)blockIdx.x * THREADS + tid; q <= g; q += (int64_t)gridDim.x * THREADS) {
            to.gIdxes[q] = from.gIdxes[q];
            if (q < g) to.nnzPerGroup[q] = from.nnzPerGroup[q];
        }
    }
}

template <int VW, bool SMALL>
__global__ __launch_bounds__(kDenseThreads) void fill_dense_blocks(const float* __restrict__ A, int64_t lda, int64_t m, int64_t k,
                                                                    int32_t p, int64_t nblk, int64_t g, DenseCounts from, DenseCounts to,
                                                                    uint32_t* __restrict__ zeroed, unsigned long long* __restrict__ ticket,
                                                                    float* __restrict__ values,
                                                                    int32_t* __restrict__ rows, int32_t* __restrict__ cols)
{
    __shared__ int32_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    place_dense_counts(from, to, g, zeroed, ticket);
    if (nblk == 0 || (int64_t)blockIdx.x >= g * nblk) return;            // the whole workgroup
    const int64_t q = blockIdx.x / nblk, b = blockIdx.x - q * nblk;      // blockIdx.x = q*nblk + b
    const int64_t c = (b * kDenseThreads + tid) * VW;
    const int64_t r0 = q * p, r1 = (r0 + p < m) ? r0 + p : m;
    const float* col0 = A + r0 * lda + c;
    uint64_t bits[VW];
    int32_t n[VW];
    if constexpr (SMALL) {
        if (c < k) {
            dense_masks<VW>(col0, lda, (int32_t)(r1 - r0), bits);
        } else {
#pragma unroll
            for (int u = 0; u < VW; ++u) bits[u] = 0;
        }
    } else {
#pragma unroll
        for (int u = 0; u < VW; ++u) n[u] = 0;
        if (c < k) {
            const float* a = col0;
            int64_t r = r0;
            for (; r + 8 <= r1; r += 8, a += 8 * lda) {
                DenseVec<VW> v[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) v[x] = load_dense<VW>(a + x * lda);
#pragma unroll
                for (int u = 0; u < VW; ++u)
#pragma unroll
                    for (int x = 0; x < 8; ++x) n[u] += (v[x].x[u] != 0.0f) ? 1 : 0;
            }
            for (; r < r1; ++r, a += lda) {
                const DenseVec<VW> v = load_dense<VW>(a);
#pragma unroll
                for (int u = 0; u < VW; ++u) n[u] += (v.x[u] != 0.0f) ? 1 : 0;
            }
        }
    }
    int32_t mine = 0;
#pragma unroll
    for (int u = 0; u < VW; ++u) {
        if constexpr (SMALL) n[u] = __popcll(bits[u]);
        mine += n[u];
    }
    int32_t incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int32_t first = from.blk[blockIdx.x].settled() + incl - mine;                  // slot of the first entry of this thread's columns
    for (int j = 0; j < w; ++j) first += wsum[j];
    if (mine == 0) return;
    int32_t at[VW];
#pragma unroll
    for (int u = 0; u < VW; ++u) { at[u] = first; first += n[u]; }
    if constexpr (SMALL) {
        while (true) {
            uint64_t any = 0;
#pragma unroll
            for (int u = 0; u < VW; ++u) any |= bits[u];
            if (!any) break;
            int32_t r[VW];
            float v[VW];
#pragma unroll
            for (int u = 0; u < VW; ++u) {
                r[u] = __ffsll((unsigned long long)bits[u]) - 1;
                if (bits[u]) v[u] = col0[r[u] * lda + u];
            }
#pragma unroll
            for (int u = 0; u < VW; ++u) {
                if (bits[u]) {
                    values[at[u]] = v[u];
                    rows[at[u]] = (int32_t)r0 + r[u];
                    cols[at[u]] = (int32_t)(c + u);
                    ++at[u];
                }
                bits[u] &= bits[u] - 1;
            }
        }
    } else {
        const float* a = col0;
        for (int64_t r = r0; r < r1; ++r, a += lda) {
            const DenseVec<VW> v = load_dense<VW>(a);
#pragma unroll
            for (int u = 0; u < VW; ++u) {
                if (v.x[u] != 0.0f) {
                    values[at[u]] = v.x[u];
                    rows[at[u]] = (int32_t)r;
                    cols[at[u]] = (int32_t)(c + u);
                    ++at[u];
                }
            }
        }
    }
}

// The same where the count left its masks behind: A is read only where it has entries.  The entries of a workgroup are listed in LDS first,
// kMaskedList at a time, so that the reads of A are in flight together and the arrays are written whole lines at a time.  Bound: the latency of the masks, the
// list and the entries in turn.  (4000 x 4000, 2 %, p = 32: 8.3 us, where fill_dense_blocks takes 19; the masks add 0.5 us to the count.)
constexpr int kMaskedList = 4096;
template <int VW>
__global__ __launch_bounds__(kDenseThreads) void fill_dense_masked(const float* __restrict__ A, int64_t lda, int64_t k, int32_t p, int64_t nblk, int64_t g,
                                                                    DenseCounts from, DenseCounts to, uint32_t* __restrict__ zeroed,
                                                                    float* __restrict__ values, int32_t* __restrict__ rows, int32_t* __restrict__ cols)
{
    static_assert(kDenseThreads * VW <= 1024, "a place in the block is listed as row * 1024 + column, in 16 bits");
    __shared__ uint16_t list[kMaskedList];
    __shared__ int32_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    place_dense_counts(from, to, g, zeroed, nullptr);
    if (nblk == 0 || (int64_t)blockIdx.x >= g * nblk) return;            // the whole workgroup
    const int64_t q = blockIdx.x / nblk, b = blockIdx.x - q * nblk;
    const int64_t c0 = b * kDenseThreads * VW, c = c0 + tid * VW, r0 = q * p;
    uint64_t bits[VW];
    int32_t mine = 0;
#pragma unroll
    for (int u = 0; u < VW; ++u) {
        bits[u] = c < k ? from.masks[q * k + c + u] : 0;
        mine += __popcll(bits[u]);
    }
    const int32_t first = from.blk[blockIdx.x].settled();
    int32_t at = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(at, d, kWave);
        if (lane >= d) at += t;
    }
    if (lane == 63) wsum[w] = at;
    __syncthreads();
    at -= mine;
    for (int j = 0; j < w; ++j) at += wsum[j];
    const int32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    const float* block = A + r0 * lda + c0;
    for (int32_t done = 0; done < total; done += kMaskedList) {
        const int32_t end = done + kMaskedList;
#pragma unroll
        for (int u = 0; u < VW; ++u) {
            while (bits[u] && at < end) {
                list[at - done] = (uint16_t)(((__ffsll((unsigned long long)bits[u]) - 1) << 10) | (tid * VW + u));
                bits[u] &= bits[u] - 1;
                ++at;
            }
        }
        __syncthreads();
        const int32_t n = total - done < kMaskedList ? total - done : kMaskedList;
#pragma unroll 4
        for (int32_t e = tid; e < n; e += kDenseThreads) {
            const int32_t r = list[e] >> 10, cc = list[e] & 1023;
            const int64_t to_slot = (int64_t)first + done + e;
            values[to_slot] = block[r * lda + cc];
            rows[to_slot] = (int32_t)r0 + r;
            cols[to_slot] = (int32_t)c0 + cc;
        }
        __syncthreads();
    }
}

// The same and the entries in row order for a matrix of up to kDenseWindow columns, `split` workgroups per group, each with a part of the columns: what a sort of the group by row would find follows from
// the masks as well.  The entries of the group, as a bit per row and column in LDS, say how many of its row lie in front of each; where the part's entries fit, they are put into row order
// there and written whole lines at a time.
// `parts`, for the band schedule: the columns of each group as a bitmap; those of a group that lies across the border of two blocks of `block_rows` rows, of no more than one, as two, the rows of the later block b
// in parts[g + b].  `places`: the long rows are listed in places of their group (RowsArgs), else by a later launch, since this one clears their count, and zeroed[kSoonWord] (FillArgs::soon).
// Bound: a chain of latencies (masks, list, entries behind the L2), a third of it the loops over a thread's bits and the sums, 16 waves side by side.  Two workgroups to a compute unit, hence 64 registers.
// Conversion with its count (us; fill, sort by row and, for bands, the bitmaps as launches of their own, and so): 4000 x 4000, 2 %: 48.7 46.9; 10 %: 83.2 65.1; 1000 x 1000, 2 %: 24.0 22.2; 300 x 300, 5 %: 23.1 21.0;
// 500 x 4000, 20 %: 78.9 47.3; 6000 x 3000, 20 %: 168 123; 14000 x 4000, 0.5 %: 83.8 83.1; 20 %: 517 352.
constexpr int kSoonWord = 28;                        // (zeroed[0] is 16 bytes behind the beginning of a line)
constexpr int kDenseGroupThreads = 1024, kDenseWindow = 4 * kDenseGroupThreads;
constexpr int dense_group_list(int rows) { return rows <= 32 ? 4096 : 2048; }      // entries that a workgroup has in LDS at a time
template <int ROWS, bool SPLIT>
__global__ __launch_bounds__(kDenseGroupThreads, 8) void fill_dense_groups(const float* __restrict__ A, int64_t lda, int64_t m, int64_t k, int32_t p, int64_t g,
                                                                         DenseCounts from, DenseCounts to, uint32_t* __restrict__ zeroed,
                                                                         float* __restrict__ values, int32_t* __restrict__ rows, int32_t* __restrict__ cols,
                                                                         RowsOut out, bool places, uint32_t* __restrict__ parts, int32_t block_rows, int32_t split)
{
    constexpr int THREADS = kDenseGroupThreads, WAVES = THREADS / kWave, WORDS = kDenseWindow / 32, PITCH = WORDS + 1;      // (a word more keeps the rows on different banks)
    constexpr int LIST = dense_group_list(ROWS), EACH = LIST / THREADS;
    constexpr int PER_ROW = THREADS / ROWS, PER_THREAD = WORDS / PER_ROW;      // threads that count a row, words of it for each
    static_assert(WAVES == 16, "");
    typedef typename std::conditional<ROWS == 32, uint32_t, uint64_t>::type Mask;
    __shared__ uint32_t bits_s[ROWS * PITCH], list[LIST];
    typedef typename std::conditional<SPLIT, uint32_t, uint16_t>::type Place;
    __shared__ Place staged_s[LIST];                          // SPLIT: as in `list`, else the column
    __shared__ uint16_t before_s[ROWS * WORDS];               // entries of the row in front of a word
    __shared__ int32_t wsum[WAVES], row_n[ROWS], row_to[ROWS];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    place_dense_counts<THREADS>(from, to, g, zeroed, nullptr);
    if (blockIdx.x == 0 && threadIdx.x == 4) zeroed[kSoonWord] = 0u;
    const int64_t q = SPLIT ? blockIdx.x / split : blockIdx.x, r0 = q * p;
    const int32_t part = SPLIT ? (int32_t)(blockIdx.x - q * split) : 0;
    const int32_t nr = (int32_t)(m - r0 < p ? m - r0 : p), g0 = from.gIdxes[q], g1 = from.gIdxes[q + 1];
    Mask bits[4];                                             // of the thread's columns, four side by side
    int32_t mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) bits[u] = 4 * tid + u < k ? (Mask)from.masks[q * k + 4 * tid + u] : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) mine += ROWS == 32 ? __popc((uint32_t)bits[u]) : __popcll(bits[u]);
    const int32_t incl = lanes_scan<64>(mine);
    if (lane == 63) wsum[w] = incl;
    for (int i = tid; i < ROWS * PITCH; i += THREADS) bits_s[i] = 0u;
    __syncthreads();
    // The workgroup's part of the columns: those of the waves [w0, w1), 256 each.
    const int32_t each = ((int32_t)((k + 255) / 256) + split - 1) / split, w0 = !SPLIT ? 0 : part * each < WAVES ? part * each : WAVES, w1 = !SPLIT ? WAVES : w0 + each < WAVES ? w0 + each : WAVES;
    const int32_t waves = lanes_scan<16>(wsum[lane & 15]);
    auto upto = [&](int32_t wave) { return wave > 0 ? __builtin_amdgcn_readlane(waves, wave - 1) : 0; };
    const int32_t before = SPLIT ? upto(w0) : 0, total = upto(w1) - before, begin = incl - mine + upto(w) - before;      // of the part, of the thread's entries in it
    // The entries `done` to done + LIST, column by column: row, and column.  The first time each leaves its bit for the row.
    auto place = [&](int32_t done, bool first) {
        int32_t at = begin - done;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (Mask b = bits[u]; b; b &= b - 1, ++at) {
                const uint32_t r = (uint32_t)(ROWS == 32 ? __ffs((uint32_t)b) : __ffsll((unsigned long long)b)) - 1u;
                if (first) atomicOr(&bits_s[r * PITCH + tid / 8], 1u << ((4 * tid + u) & 31));
                if ((!SPLIT || (w >= w0 && w < w1)) && (uint32_t)at < (uint32_t)LIST) list[at] = r * kDenseWindow + (uint32_t)(4 * tid + u);
            }
    };
    place(0, true);
    __syncthreads();
    const bool staged = total <= LIST;                        // the row order goes through LDS and out in whole lines
    const float* band = A + r0 * lda;
    int32_t row_at = 0, row_from = 0;                         // of row `lane`: its place in the row order, what takes a place in it to one in the staged part
    for (int32_t done = 0; done < total || done == 0; done += LIST) {
        const int32_t n = total - done < LIST ? total - done : LIST;
        float v[EACH];
        uint32_t e[EACH];
        if (done > 0) {
            __syncthreads();
            place(done, false);
            __syncthreads();
        }
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            e[x] = x * THREADS + tid < n ? list[x * THREADS + tid] : 0u;
            v[x] = n > 0 ? band[(int64_t)(e[x] / kDenseWindow) * lda + e[x] % kDenseWindow] : 0.0f;
        }
        if (done == 0) {                                      // (while the values are on their way)
            const int r = tid / PER_ROW, j = tid % PER_ROW;
            int32_t in_front[PER_THREAD], sum = 0;
#pragma unroll
            for (int x = 0; x < PER_THREAD; ++x) {
                in_front[x] = sum;
                sum += __popc(bits_s[r * PITCH + j * PER_THREAD + x]);
            }
            const int32_t so_far = lanes_scan<PER_ROW>(sum);
            const int32_t word = tid - (THREADS - WORDS), nbw = (int32_t)((k + 31) / 32);
            if (parts && part == 0 && word >= 0 && word < nbw) {
                const int64_t later = r0 / block_rows + 1;
                const int32_t mid = later * block_rows - r0 < nr ? (int32_t)(later * block_rows - r0) : nr;
                uint32_t here = 0u, beyond = 0u;
#pragma unroll 4
                for (int i = 0; i < ROWS; ++i) (i < mid ? here : beyond) |= bits_s[i * PITCH + word];
                parts[q * nbw + word] = here;
                if (mid < nr) parts[(g + later) * nbw + word] = beyond;
            }
#pragma unroll
            for (int x = 0; x < PER_THREAD; ++x) before_s[r * WORDS + j * PER_THREAD + x] = (uint16_t)(so_far - sum + in_front[x]);
            if (j == PER_ROW - 1) row_n[r] = so_far;
            __syncthreads();
            const int32_t of_row = lane < ROWS ? row_n[lane] : 0;
            row_at = g0 + lanes_scan<64>(of_row) - of_row;
            if constexpr (SPLIT) {
                const int32_t skip = lane < ROWS && w0 > 0 ? (w0 < WAVES ? (int32_t)before_s[lane * WORDS + 8 * w0] : of_row) : 0;
                const int32_t here = (lane < ROWS && w1 < WAVES ? (int32_t)before_s[lane * WORDS + 8 * w1] : of_row) - skip;
                row_from = lanes_scan<64>(here) - here - skip;
                if (w == 0 && lane < ROWS) row_to[lane] = row_at - row_from;
            } else {
                row_from = row_at - g0;
            }
            if (w == 0 && part == 0) {
                if (lane < nr) out.start[r0 + lane] = row_at;
                if (lane == 0 && q == g - 1) out.start[m] = g1;
                if (places) {
                    // as in order_groups: a group has the places that the multiples of long_row in its stretch give it, never fewer than rows of more entries than that
                    const int32_t l0 = g0 / out.long_row, l1 = g1 / out.long_row;
                    const uint64_t is = __ballot(lane < nr && of_row > out.long_row);
                    const int32_t at = l0 + __popcll(is & lanemask_lt());
                    if ((is >> lane & 1) && at < l1) out.long_rows[at] = (int32_t)r0 + lane;
                    for (int32_t i = l0 + __popcll(is) + lane; i < l1; i += kWave) out.long_rows[i] = -1;
                }
            }
        }
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            const uint32_t r = e[x] / kDenseWindow, c = e[x] % kDenseWindow;
            const int32_t by_row = __shfl(staged ? row_from : row_at, (int)r, kWave) + (int32_t)before_s[r * WORDS + c / 32] + __popc(bits_s[r * PITCH + c / 32] & ((1u << (c & 31u)) - 1u));
            if (x * THREADS + tid < n) {
                const int32_t slot = g0 + before + done + x * THREADS + tid;
                values[slot] = v[x];
                rows[slot] = (int32_t)(r0 + r);
                cols[slot] = (int32_t)c;
                if (staged) {
                    list[by_row] = __float_as_uint(v[x]);
                    staged_s[by_row] = (Place)(SPLIT ? e[x] : c);
                } else {
                    out.cols[by_row] = (int32_t)c;
                    out.vals[by_row] = v[x];
                }
            }
        }
    }
    if (staged) {
        __syncthreads();
        for (int32_t i = tid; i < total; i += THREADS) {
            const uint32_t e = staged_s[i];
            const int32_t to_slot = (SPLIT ? row_to[e / kDenseWindow] : g0) + i;
            out.cols[to_slot] = (int32_t)(e % kDenseWindow);
            out.vals[to_slot] = __uint_as_float(list[i]);
        }
    }
}

// Total count of entries != 0 of a dense matrix (Algorithm 1, step 1, without the grouping): pieces of 16 rows x kDenseThreads*VW
// columns, strided over the workgroups.
template <int VW>
__global__ __launch_bounds__(kDenseThreads) void count_dense_total(const float* __restrict__ A, int64_t lda, int64_t m, int64_t k, int64_t nblk,
                                                                    DenseTicket ticket, unsigned long long* __restrict__ host)
{
    constexpr int64_t ROWS = 16;
    __shared__ unsigned long long wide[4];
    unsigned long long n = 0;
    const int64_t items = (m + ROWS - 1) / ROWS * nblk;
    for (int64_t i = blockIdx.x; i < items; i += gridDim.x) {
        const int64_t q = i / nblk, b = i - q * nblk;
        const int64_t c = (b * kDenseThreads + threadIdx.x) * VW;
        const int64_t r0 = q * ROWS, r1 = (r0 + ROWS < m) ? r0 + ROWS : m;
        if (c < k) n += (unsigned long long)count_dense_tile<VW>(A, lda, r0, r1, c);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_down(n, d, kWave);
    if ((threadIdx.x & 63) == 0) wide[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long all;
        if (arrive(ticket, wide[0] + wide[1] + wide[2] + wide[3], &all)) {   // integer sum: order-free
            wait_for_memory();
            tell_host(host, all);
        }
    }
}

}  // namespace gcoo
