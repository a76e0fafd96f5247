// Conversion of a CSR input without a sort, in two kernels or one: take_rows reads the input once, order_groups writes the five arrays, or does both.
//
// Inside a group the entries are ordered by (column, row).  With the rows that hold an entry in a column as a bit mask per
// column (at most p bits), the place of an entry is what the columns before it hold, a prefix sum of popcounts, plus the
// popcount of the mask below its row: two passes over the entries with a few LDS accesses each, no ranking, any order inside the rows.
// The radix sort (gcoo_build_kernels.hpp) moves every entry through memory once per digit and walks it in tiles of 64
// with eight ballots each; it stays for matrices whose columns far outnumber the entries of a group (more than 128 to one; order_plan() in gcoo_api.hip).
//
// A workgroup orders one part of a group: `ncols` columns.  Where the columns of every row ascend, which take_rows checks, a part is
// one stretch of each row, and take_rows has noted where it begins; otherwise the workgroup looks through the whole group.
// A group that holds a coordinate twice has no place for it in a mask: such a part is ranked in input order by one wave.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gcoo_band_build.hpp"
#include "gcoo_build_kernels.hpp"

namespace gcoo {

constexpr int kOrderThreads = 256;
constexpr int kOrderMaxParts = 64;
constexpr int kOrderMaxCap = 3072;       // entries of a part that are put in order in LDS; a larger part is written in place
constexpr uint32_t kBadColumn = 1u, kUnsorted = 2u, kHeavy = 4u;

// How the groups of a matrix are cut; the same on the host for the layout and for the launches.
struct OrderPlan {
    int32_t shift;             // log2 of the columns of a part
    int32_t parts;
    int32_t list_rows;         // rows per workgroup of take_rows
    int32_t cap;
    bool fused;
    int32_t keys;              // 0, or ranked: distinct columns of a window
    int32_t threads;           // of a workgroup of order_groups
    bool both;                 // order_groups and band_fill are one launch
};

struct TakeArgs {
    const int32_t* row_ptr;
    const int32_t* cols;
    const float* vals;
    int64_t m, g, lists;
    int32_t p, nnz, k;
    OrderPlan plan;
    int32_t* gIdxes;
    int32_t* nnzPerGroup;
    int32_t* row_start;        // [m + 1]
    int32_t* row_cols;         // entries in row order, or null
    float* row_vals;
    uint32_t* flags;           // [lists]
    int32_t* splits;           // [m * (parts - 1)] where the later parts of a row begin
    uint32_t* bits;            // [lists * ceil(k/32)] columns of a list, or null
    int32_t heavy;             // a list of more entries makes the matrix uneven
    uint32_t* zero_bad;        // bad_col, the count of long rows, the word for uneven matrices, the count of the longest rows
    unsigned long long* stats; // or null; a workgroup more
};

// Row r with start[r] <= e < start[r + 1], among ascending starts of which those from the last row's end on are INT32_MAX; empty
// rows are skipped.  Always log2(ROWS) steps, so that a thread's entries go through it side by side.
template <int ROWS>
__device__ __forceinline__ int32_t row_of_entry(const int32_t* start, int32_t e)
{
    int32_t r = 0;
#pragma unroll
    for (int d = ROWS / 2; d >= 1; d >>= 1) r += start[r + d] <= e ? d : 0;
    return r;
}

// One workgroup per list of rows.  Bound: memory, an entry is read once and its copy in row order written once.  Dynamic LDS: the
// list's columns as a bitmap, where the band schedule wants it.  FROM kTakeHost: the input is host memory, and a column is not read twice
// (from device memory the second read, which the vector cache serves, is the cheaper way: 36.6 and 42.7 us for 6.4 million entries).  kTakeHost16: its columns have 16 bits (TakeArgs::cols points to
// them), six bytes per entry over the link in place of eight (conversion and product, us, eight and six: 3881 x 4000, 1.28 %, N = 516: 77.8 70.6; 2877 x 3824, 1.29 %, N = 1183: 77.0 71.8).
// THREADS = 1024 for lists of more than 2048 entries, of which there are few (4000 x 4000, 5 %: 10.0 us with 512, 8.4 so; 8000 x 8000, 10 %: 24.2 and 23.0; but
// 0.5 %: 6.6 and 7.3; before the rows were found by lanes 10.0 and 27.6 for the first two).
enum TakeFrom { kTakeDevice, kTakeHost, kTakeHost16 };
template <TakeFrom FROM, int THREADS>
__global__ __launch_bounds__(THREADS) void take_rows(TakeArgs a)
{
    constexpr int EACH = 4;
    auto column = [&](int32_t e) -> int32_t { return FROM == kTakeHost16 ? (int32_t)reinterpret_cast<const uint16_t*>(a.cols)[e] : a.cols[e]; };
    extern __shared__ uint32_t take_bits[];
    __shared__ int32_t rs[66];
    __shared__ uint32_t flag_s;
    const int tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x == a.lists) {                                 // the whole workgroup
        group_stats_block<THREADS>(a.row_ptr, a.m, a.p, a.g, a.stats);
        return;
    }
    const int32_t list = (int32_t)blockIdx.x;
    if (list == 0 && tid < 4) a.zero_bad[tid] = 0u;
    // Offsets are clamped to [0, nnz]: with a device input whose row_ptr does not match the nnz the buffer was laid out
    // for, every later kernel still stays inside the arrays.
    const int32_t nnz = a.nnz, m = (int32_t)a.m;
    auto at = [&](int32_t r) { const int32_t v = a.row_ptr[r]; return v < 0 ? 0 : (v > nnz ? nnz : v); };
    const int32_t r0 = (int64_t)list * a.plan.list_rows < m ? list * a.plan.list_rows : m;
    const int32_t rows = m - r0 < a.plan.list_rows ? m - r0 : a.plan.list_rows;
    const int32_t nbw = (a.k + 31) / 32;
    if (tid == 0) flag_s = 0u;
    if (tid <= rows) {
        const bool group = tid < rows && (uint32_t)(r0 + tid) % (uint32_t)a.p == 0;
        const int32_t v = at(r0 + tid), next = group ? at(a.p < m - (r0 + tid) ? r0 + tid + a.p : m) : 0;
        rs[tid] = v;
        a.row_start[r0 + tid] = v;
        if (group) {
            const int32_t q = (int32_t)((uint32_t)(r0 + tid) / (uint32_t)a.p);
            a.gIdxes[q] = v;
            a.nnzPerGroup[q] = next < v ? 0 : next - v;
        }
        if (r0 + tid == m) a.gIdxes[a.g] = v;
    }
    if (a.bits)
        for (int32_t i = tid; i < nbw; i += THREADS) take_bits[i] = 0u;
    __syncthreads();
    const int32_t shift = a.plan.shift, later = a.plan.parts - 1;
    uint32_t flag = 0u;
    if (tid < rows) {
        const int32_t b = rs[tid];
        if (rs[tid + 1] < b) flag |= kUnsorted;                  // offsets that contradict each other
        if (rs[tid + 1] <= b)
            for (int32_t j = 0; j < later; ++j) a.splits[(int64_t)(r0 + tid) * later + j] = b;
    }
    const int32_t beg = rs[0], end = rs[rows], start = lane < rows ? rs[lane] : INT32_MAX;
    auto in_range = [&](int32_t c) { return c < 0 ? 0 : (c >= a.k ? a.k - 1 : c); };
    for (int32_t e = beg + tid; e - tid < end; e += EACH * THREADS) {       // (the whole wave)
        int32_t c[EACH], before[EACH];
        float v[EACH];
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            const int32_t i = e + x * THREADS < end ? e + x * THREADS : end - 1;
            c[x] = column(i);
            if (a.row_cols) v[x] = a.vals[i];
            // the column before it
            if constexpr (FROM != kTakeDevice) {
                const int32_t first = (tid & 63) == 0 && i > beg ? column(i - 1) : 0;
                before[x] = __builtin_amdgcn_update_dpp(first, c[x], 0x138, 0xf, 0xf, false);       // wave_shr:1
            } else {
                before[x] = a.cols[i > beg ? i - 1 : i];
            }
        }
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            // The entry's row, and whether it is its first and its last: the rows that begin up to the entry of the wave's first lane, and those
            // that begin at the 64 behind it, from the lanes, which hold where the rows begin (a search in LDS reads six words one after another).
            const int32_t i = e + x * THREADS < end ? e + x * THREADS : end - 1, i0 = __builtin_amdgcn_readfirstlane(i);
            const uint64_t here = __ballot(start == i0);                         // (of all lanes)
            int32_t r = __popcll(__ballot(start <= i0)) - 1;
            bool first = i == i0 && here != 0, last = i + 1 == end;
            for (uint64_t in = __ballot(start > i0 && start - i0 <= 64); in; in &= in - 1) {
                const int32_t begins = __builtin_amdgcn_readlane(start, __ffsll((unsigned long long)in) - 1);
                r += begins <= i;
                first |= begins == i;
                last |= begins == i + 1;
            }
            if (e + x * THREADS < end) {
                const int32_t col = in_range(c[x]), prev = in_range(before[x]);
                if (col != c[x]) flag |= kBadColumn;
                if (!first && prev >= col) flag |= kUnsorted;
                if (a.row_cols) {
                    a.row_cols[i] = col;
                    a.row_vals[i] = v[x];
                }
                if (a.bits) atomicOr(&take_bits[col >> 5], 1u << (col & 31));
                if (later > 0) {
                    int32_t* split = a.splits + (int64_t)(r0 + r) * later - 1;
                    const int32_t part = col >> shift;
                    for (int32_t j = first ? 1 : (prev >> shift) + 1; j <= part; ++j) split[j] = i;
                    if (last)
                        for (int32_t j = part + 1; j <= later; ++j) split[j] = i + 1;
                }
            }
        }
    }
    if (flag) atomicOr(&flag_s, flag);
    __syncthreads();
    if (tid == 0) a.flags[list] = flag_s | (end - beg > a.heavy ? kHeavy : 0u);
    if (a.bits)
        for (int32_t i = tid; i < nbw; i += THREADS) a.bits[(int64_t)list * nbw + i] = take_bits[i];
}

struct OrderArgs {
    const int32_t* row_start;
    const int32_t* cols;       // entries in row order; clamped here
    const float* vals;
    int64_t m, lists;
    int32_t p, k;
    OrderPlan plan;
    const int32_t* gIdxes;
    const uint32_t* flags;
    const int32_t* splits;
    RowsOut out;               // long rows
    uint32_t* uneven;          // set where a list is heavy
    int32_t* dst_cols;
    int32_t* dst_rows;
    float* dst_vals;
    // FUSED only: the input's offsets, and what take_rows would have written
    const int32_t* row_ptr;
    int32_t nnz;
    int64_t g;
    int32_t* gIdxes_out;
    int32_t* nnzPerGroup_out;
    int32_t* row_start_out;
    uint32_t* flags_out;       // [g]
    bool far;                  // the input is in host memory
};

inline size_t order_lds_bytes(const OrderPlan& plan, int words)
{
    if (plan.keys) return ((size_t)2 << plan.shift) / 8 + (size_t)plan.keys * (4 * words + 4) + (size_t)plan.cap * 8;
    const size_t ncols = (size_t)1 << plan.shift, spare = ncols < (size_t)plan.threads ? ncols : (size_t)plan.threads;
    return (ncols * (words + 1) + 2 * spare) * 4 + (size_t)plan.cap * 8;
}

// Workgroup (q, part).  WORDS = 32-bit words of a column's mask.  Dynamic LDS: order_lds_bytes().
// Bound: the latency of the chain of steps.  A thread takes eight entries through each step side by side and keeps them between the
// two passes where they are all, the parts are small enough for several workgroups per compute unit, and a part's entries leave LDS in
// their order, so that the stores are whole lines.
// (Index, two radix passes and bitmaps before, take_rows and this now: 8000 x 8000, 10 %: 190 -> 78 us; 0.5 %: 28 -> 17; 4000 x 4000,
// 5 %: 41 -> 19; power-law rows, 16384 x 16384: 65 -> 40.  The sums over a workgroup by DPP and one barrier each, here and in band_fill_list(), instead of shuffles and up to 16 reads of LDS, conversion and
// product: 1777 x 2301, 3 %, N = 1117: 33.3 32.9; 4000 x 4000, 5 %: 180.8 179.3; power-law rows, 16384 x 16384, N = 512: 128.6 127.1.)
//
// FUSED (one part per group, no band schedule): there is nothing to know about a group but its rows, so this is the whole conversion, one
// launch instead of two (256 x 256: 4.2 + 6.4 us before, 6.3 so; order_plan() has more).
//
// RANKED (many columns per entry): a part has many more columns, of which a bitmap says which hold an entry; the places of those among themselves take the
// place of the columns, so that nothing is done per column but for a bit.  More distinct columns than plan.keys go window by window.
//
// HOST: as FUSED, for an input in host memory.  The launch says in the kernel's arguments where the groups begin, so that a group's entries are asked for beside its rows' starts and not one
// trip over the link behind them, and the columns have 16 bits there, six bytes per entry in place of eight: 2500 x 2500, 1 %: 17.7 -> 14.1 us, of which the link takes about 7 (9 with eight).
enum OrderKind { kOrderMasks, kOrderFused, kOrderRanked, kOrderHost };
constexpr int kOrderHostGroups = 512;        // at most, 2 KB of arguments
struct GroupStarts { int32_t at[kOrderHostGroups + 1]; };
template <int WORDS, OrderKind KIND, int THREADS>
__device__ __forceinline__ void order_part(const OrderArgs& a, int32_t item, int32_t known0 = 0, int32_t known1 = 0)
{
    constexpr int ROWS = WORDS == 8 ? 256 : 32 * WORDS, WAVES = THREADS / 64, EACH = 8;
    constexpr bool HOST = KIND == kOrderHost, FUSED = KIND == kOrderFused || HOST, RANKED = KIND == kOrderRanked;
    extern __shared__ uint32_t order_lds[];
    __shared__ int32_t seg[ROWS], off[ROWS];     // a row's place among the part's entries (or in the input), and what takes it to the input
    __shared__ int32_t wsum[WAVES], wsum2[WAVES], any_s[WAVES];
    __shared__ int32_t below_s, count_s, long_s, group_s[2];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t parts = a.plan.parts, shift = a.plan.shift, ncols = 1 << shift, later = parts - 1;
    const int64_t q = item / parts;
    const int32_t part = (int32_t)(item - q * parts);
    const int64_t r0 = q * a.p;
    const int32_t rows = (int32_t)(a.m - r0 < a.p ? a.m - r0 : a.p);
    // A thread sums up `1 << ps` columns one after another: a word more for each such stretch keeps the threads on different banks.
    constexpr int LOG = THREADS == 256 ? 8 : (THREADS == 512 ? 9 : 10);
    static_assert(THREADS == 1 << LOG, "");
    const int32_t ps = RANKED ? 31 : (shift > LOG ? shift - LOG : 0), spare = RANKED ? 0 : ((ncols - 1) >> ps) + 1;
    const int32_t nbw = ncols >> 5;                          // RANKED: words of the part's columns; how many lie in front of each word
    uint32_t* bits = order_lds;
    int32_t* before = (int32_t*)(bits + nbw);
    const int32_t keys = RANKED ? a.plan.keys : ncols;        // columns, or distinct columns of a window
    uint32_t* mask = RANKED ? (uint32_t*)(before + nbw) : order_lds;       // the masks, then the first places of the columns
    int32_t* base = (int32_t*)(mask + keys * WORDS + spare);
    float* o_val = (float*)(base + keys + spare);
    auto mask_at = [&](int32_t key) { return mask + key * WORDS + (RANKED ? 0 : key >> ps); };
    auto base_at = [&](int32_t key) { return base + key + (RANKED ? 0 : key >> ps); };
    uint32_t* o_place = (uint32_t*)(o_val + a.plan.cap);      // row | column << 8

    // everything that does not wait for anything else
    int32_t g0 = known0, g1 = known1;
    int32_t rs0 = 0, re = 0, s = 0, e = 0;
    if constexpr (FUSED) {
        // Every wave asks for the group's own offsets, so that the entries wait for nothing else; in host memory, where each would be a read over the link, one thread for all.
        auto at = [&](int64_t r) { const int32_t x = a.row_ptr[r]; return x < 0 ? 0 : (x > a.nnz ? a.nnz : x); };    // as in take_rows
        if (!HOST && !a.far) {
            g0 = at(r0);
            g1 = at(r0 + rows);
        }
        if (!HOST && a.far && tid == 0) group_s[1] = at(r0 + rows);
        if (tid < rows) {
            rs0 = at(r0 + tid);
            a.row_start_out[r0 + tid] = rs0;
        }
        if (!HOST && a.far) {
            if (tid == 0) group_s[0] = rs0;
            __syncthreads();
            g0 = __builtin_amdgcn_readfirstlane(group_s[0]);
            g1 = __builtin_amdgcn_readfirstlane(group_s[1]);
        }
        if (tid == 0) {
            a.gIdxes_out[q] = g0;
            a.nnzPerGroup_out[q] = g1 < g0 ? 0 : g1 - g0;
            if (q == a.g - 1) {
                a.gIdxes_out[a.g] = g1;
                a.row_start_out[a.m] = g1;
            }
        }
    } else {
        g0 = a.gIdxes[q];
        g1 = a.gIdxes[q + 1];
    }
    if (!FUSED && tid < rows) {
        rs0 = a.row_start[r0 + tid];
        re = a.row_start[r0 + tid + 1];
        s = part == 0 ? rs0 : a.splits[(r0 + tid) * later + part - 1];
        e = part == later ? re : a.splits[(r0 + tid) * later + part];
    }
    uint32_t f = 0u;
    if (!FUSED && (parts > 1 || a.uneven)) {
        const int64_t l0 = r0 / a.plan.list_rows, l1 = (r0 + rows - 1) / a.plan.list_rows;
        for (int64_t l = l0 + tid; l <= l1; l += THREADS) f |= a.flags[l];
        if (part == 0 && a.uneven && (f & kHeavy)) *a.uneven = 1u;
    }
    if (tid == 0) { below_s = 0; count_s = 0; long_s = 0; }
    if constexpr (RANKED) {
        for (int32_t i = tid; i < nbw; i += THREADS) bits[i] = 0u;
    } else {
        for (int32_t i = tid; i < ncols * WORDS + spare; i += THREADS) mask[i] = 0u;
    }
    // With one part the group is taken in the order of the input and nothing depends on the order in its rows.
    const bool in_order = !FUSED && parts > 1 && !block_any<WAVES>((f & kUnsorted) != 0, any_s);
    const bool some = !FUSED && parts > 1 && !in_order;                // entries of other parts are among those looked at

    int32_t n = FUSED ? g1 - g0 : 0, out0 = FUSED ? g0 : 0;  // entries to look at, place of the part's first one in the arrays
    const int32_t c0 = part << shift, kmax = a.k - 1, wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    bool bad = false;                                        // FUSED: a column was out of range
    // Entry i of those to look at is of row r, in column c of the part.  A thread goes through eight at a time, side by side, past the end the last one again; a wave that has no more than four
    // per thread goes through four: what is past the end costs a search and two requests as well (conversion and product, us, eight always and so: 1777 x 2301, 3 %, N = 1117: 35.4 34.6; power-law
    // rows, 16384 x 16384, N = 512: 140.6 134.8; one, two, four or eight: 34.5 and 139, and twice the code).
    static_assert(EACH == 8, "four and four");
    int32_t r[EACH], c[EACH];
    float v[EACH];
    auto column = [&](int32_t at) -> int32_t { return HOST ? (int32_t)reinterpret_cast<const uint16_t*>(a.cols)[at] : a.cols[at]; };
    auto inside = [&](int32_t col) { return col < 0 ? 0 : (col > kmax ? kmax : col); };
    auto ask = [&](auto from, int32_t i0) {
#pragma unroll
        for (int x = decltype(from)::value; x < decltype(from)::value + 4; ++x) {
            const int32_t i = i0 + x * THREADS + tid, e = i < n ? i : n - 1;
            if constexpr (!FUSED) r[x] = row_of_entry<ROWS>(seg, e);
            const int32_t at = FUSED ? g0 + e : off[r[x]] + e;
            c[x] = column(at);
            v[x] = a.vals[at];
        }
    };
    auto find = [&](auto from, int32_t i0) {
#pragma unroll
        for (int x = decltype(from)::value; x < decltype(from)::value + 4; ++x) {
            const int32_t i = i0 + x * THREADS + tid, col = c[x];
            if constexpr (FUSED) {
                r[x] = row_of_entry<ROWS>(seg, g0 + (i < n ? i : n - 1));
                bad |= inside(col) != col;
            }
            c[x] = inside(col) - c0;
        }
    };
    auto take = [&](int32_t i, int32_t* ri, int32_t* ci, float* vi) {
        *ri = row_of_entry<ROWS>(seg, FUSED ? g0 + i : i);
        const int32_t at = FUSED ? g0 + i : off[*ri] + i;
        *ci = inside(column(at)) - c0;
        *vi = a.vals[at];
    };
    if constexpr (FUSED) {
        if (wave0 < n) {
            ask(std::integral_constant<int, 0>{}, 0);
            if (n - wave0 > 4 * THREADS) ask(std::integral_constant<int, 4>{}, 0);
        }
    }
    if (in_order) {
        const int32_t len = e - s;
        const int32_t at = block_scan<WAVES>(len, wsum, &n);
        int32_t skip;
        block_scan<WAVES>(s - rs0, wsum2, &skip);
        out0 = g0 + skip;
        if (tid < ROWS) {
            seg[tid] = tid < rows ? at : INT32_MAX;
            off[tid] = s - at;
        }
    } else if (FUSED) {
        if (tid < ROWS) seg[tid] = tid < rows ? rs0 : INT32_MAX;       // (in the input)
    } else {
        n = g1 - g0;
        out0 = g0;
        if (tid < ROWS) {
            seg[tid] = tid < rows ? rs0 - g0 : INT32_MAX;
            off[tid] = g0;
        }
    }
    __syncthreads();
    if (!FUSED && part == 0 && tid < rows && a.out.cols) list_long_row(a.out, (int32_t)r0 + tid, re - rs0);
    if (n <= 0) {                                            // the whole workgroup
        if (FUSED && tid == 0) a.flags_out[q] = 0u;
        return;
    }
    // FUSED: no earlier launch has cleared a count of long rows, so a group has places of its own among them, those that the multiples of long_row
    // in its stretch of the entries give it: never fewer than it has rows of more entries than that.
    int32_t long0 = 0, long1 = 0;
    if (FUSED && a.out.cols) {
        long0 = g0 / a.out.long_row;
        long1 = g1 / a.out.long_row;
        if (tid < rows && (tid + 1 < rows ? seg[tid + 1] : g1) - seg[tid] > a.out.long_row) {
            const int32_t at = long0 + atomicAdd(&long_s, 1);
            if (at < long1) a.out.long_rows[at] = (int32_t)r0 + tid;
        }
    }
    auto take_some = [&](int32_t i0, bool asked = false) {
        const int32_t left = n - i0 - wave0;                 // from the wave's first entry on
        if (left <= 0) return;
        if (!asked) ask(std::integral_constant<int, 0>{}, i0);
        if (left > 4 * THREADS) {
            if (!asked) ask(std::integral_constant<int, 4>{}, i0);
            find(std::integral_constant<int, 4>{}, i0);
        }
        find(std::integral_constant<int, 0>{}, i0);
    };

    // the masks (RANKED: the bitmap); what lies before the part and what is in it, where that is not known yet
    bool twice = false;
    int32_t below = 0, mine = 0;
    for (int32_t i0 = 0; i0 < n; i0 += EACH * THREADS) {
        take_some(i0, FUSED && i0 == 0);
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            if (i0 + x * THREADS + tid >= n) break;
            if (some) {
                below += c[x] < 0;
                if (c[x] < 0 || c[x] >= ncols) continue;
                ++mine;
            }
            if (FUSED && a.out.cols) {                       // the entries in row order
                a.out.cols[g0 + i0 + x * THREADS + tid] = c[x];
                a.out.vals[g0 + i0 + x * THREADS + tid] = v[x];
            }
            if constexpr (RANKED) {
                atomicOr(&bits[c[x] >> 5], 1u << (c[x] & 31));
            } else {
                const uint32_t bit = 1u << (r[x] & 31);
                const uint32_t old = atomicOr(mask_at(c[x]) + (r[x] >> 5), bit);
                twice |= (old & bit) != 0;
            }
        }
    }
    int32_t count = n;
    if (some) {
        if (below) atomicAdd(&below_s, below);
        if (mine) atomicAdd(&count_s, mine);
    }
    if (FUSED && bad) atomicOr(&below_s, 1);
    if (!RANKED) twice = block_any<WAVES>(twice, any_s);
    else __syncthreads();
    if (FUSED && tid == 0) a.flags_out[q] = below_s ? kBadColumn : 0u;
    if (FUSED)
        for (int32_t i = long0 + long_s + tid; i < long1; i += THREADS) a.out.long_rows[i] = -1;
    if (some) {
        out0 = g0 + below_s;
        count = count_s;
        if (count == 0) return;                              // the whole workgroup
    }
    // (wsum was read before the barrier above, or the one at the end here)
    auto prefix = [&](int32_t x, int32_t* all) { return block_scan<WAVES>(x, wsum, all); };
    int32_t distinct = ncols;
    if constexpr (RANKED) {
        const int32_t per = (nbw + THREADS - 1) / THREADS, i0 = tid * per < nbw ? tid * per : nbw, i1 = i0 + per < nbw ? i0 + per : nbw;
        int32_t sum = 0;
        for (int32_t i = i0; i < i1; ++i) sum += __popc(bits[i]);
        int32_t at = prefix(sum, &distinct);
        for (int32_t i = i0; i < i1; ++i) {
            before[i] = at;
            at += __popc(bits[i]);
        }
    }
    const bool staged = count <= a.plan.cap && (!RANKED || distinct <= keys);
    for (int32_t w0 = 0; w0 < distinct; w0 += keys) {        // (one turn where a window holds all, always so without RANKED)
        const int32_t nk = distinct - w0 < keys ? distinct - w0 : keys;
        // what stands for a column: itself, or its place among the distinct ones of the window
        auto key_of = [&](int32_t col) -> int32_t {
            if (!RANKED) return col;
            return before[col >> 5] + __popc(bits[col >> 5] & ((1u << (col & 31)) - 1u)) - w0;
        };
        auto ours = [&](int32_t col) { return !some || (col >= 0 && col < ncols); };
        int32_t key[EACH];
        if constexpr (RANKED) {
            for (int32_t i = tid; i < nk * WORDS; i += THREADS) mask[i] = 0u;
            __syncthreads();
            twice = false;
            for (int32_t i0 = 0; i0 < n; i0 += EACH * THREADS) {
                if (n > EACH * THREADS) take_some(i0);
#pragma unroll
                for (int x = 0; x < EACH; ++x) key[x] = i0 + x * THREADS + tid < n && ours(c[x]) ? key_of(c[x]) : -1;
#pragma unroll
                for (int x = 0; x < EACH; ++x) {
                    if (key[x] < 0 || key[x] >= nk) continue;
                    const uint32_t bit = 1u << (r[x] & 31);
                    const uint32_t old = atomicOr(mask_at(key[x]) + (r[x] >> 5), bit);
                    twice |= (old & bit) != 0;
                }
            }
            twice = block_any<WAVES>(twice, any_s);
        }
        if (twice) {
            // counts instead of masks
            for (int32_t i = tid; i < keys + spare; i += THREADS) base[i] = 0;
            __syncthreads();
            for (int32_t i = tid; i < n; i += THREADS) {
                int32_t ri, ci;
                float vi;
                take(i, &ri, &ci, &vi);
                const int32_t ki = ours(ci) ? key_of(ci) : -1;
                if (ki >= 0 && ki < nk) atomicAdd(base_at(ki), 1);
            }
            __syncthreads();
        }
        // the first place of every column
        int32_t entries_of_window;
        {
            const int32_t per = RANKED ? (nk + THREADS - 1) / THREADS : 1 << ps;
            const int32_t i0 = RANKED ? (tid * per < nk ? tid * per : nk) : tid << ps, i1 = i0 + per < nk ? i0 + per : nk;
            auto entries = [&](int32_t k) {
                if (twice) return *base_at(k);
                int32_t x = 0;
#pragma unroll
                for (int w = 0; w < WORDS; ++w) x += __popc(mask_at(k)[w]);
                return x;
            };
            int32_t sum = 0, kept[4];
            if (per <= 4) {                                  // (the same for all)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    kept[x] = sum;
                    if (i0 + x < i1) sum += entries(i0 + x);
                }
                const int32_t at = prefix(sum, &entries_of_window);
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (i0 + x < i1) *base_at(i0 + x) = at + kept[x];
            } else {
#pragma unroll 4
                for (int32_t i = i0; i < i1; ++i) sum += entries(i);
                int32_t at = prefix(sum, &entries_of_window);
#pragma unroll 4
                for (int32_t i = i0; i < i1; ++i) {
                    const int32_t x = entries(i);
                    *base_at(i) = at;
                    at += x;
                }
            }
        }
        __syncthreads();
        if (twice) {
            // 64 entries at a time, in input order
            for (int32_t t = 0; t < n && wv == 0; t += 64) {
                int32_t ri = 0, ci = -1;
                float vi = 0.0f;
                if (t + lane < n) take(t + lane, &ri, &ci, &vi);
                const int32_t ki = t + lane < n && ci >= 0 && ci < ncols ? key_of(ci) : -1;
                const bool act = ki >= 0 && ki < nk;
                uint64_t same = __ballot(act);
                for (int b = 0; (keys - 1) >> b; ++b) {
                    const bool bit = (ki >> b) & 1;
                    const uint64_t bb = __ballot(act && bit);
                    same &= bit ? bb : ~bb;
                }
                const int32_t ahead = __popcll(same & lanemask_lt());
                int32_t slot = 0;
                volatile int32_t* next = base_at(act ? ki : 0);
                if (act) slot = *next;
                __builtin_amdgcn_wave_barrier();
                if (act && ahead == 0) *next = slot + __popcll(same);
                __builtin_amdgcn_wave_barrier();
                if (act) {
                    const int32_t to = out0 + slot + ahead;
                    a.dst_cols[to] = c0 + ci;
                    a.dst_rows[to] = (int32_t)r0 + ri;
                    a.dst_vals[to] = vi;
                }
            }
        } else {
            for (int32_t i0 = 0; i0 < n; i0 += EACH * THREADS) {
                if (n > EACH * THREADS) take_some(i0);         // (else they are still there)
#pragma unroll
                for (int x = 0; x < EACH; ++x) {
                    if (i0 + x * THREADS + tid >= n) break;
                    if (!ours(c[x])) continue;
                    const int32_t ki = RANKED && n <= EACH * THREADS ? key[x] : key_of(c[x]);
                    if (RANKED && (ki < 0 || ki >= nk)) continue;
                    int32_t at = *base_at(ki);
#pragma unroll
                    for (int w = 0; w < WORDS; ++w) {
                        const uint32_t word = mask_at(ki)[w];
                        const int32_t b = r[x] - 32 * w;
                        at += __popc(WORDS == 1 || b < 32 ? (b <= 0 ? 0u : word & ((1u << b) - 1u)) : word);
                    }
                    if (staged) {
                        o_val[at] = v[x];
                        o_place[at] = (uint32_t)r[x] | (uint32_t)c[x] << 8;
                    } else {
                        a.dst_cols[out0 + at] = c0 + c[x];
                        a.dst_rows[out0 + at] = (int32_t)r0 + r[x];
                        a.dst_vals[out0 + at] = v[x];
                    }
                }
            }
            if (staged) {
                __syncthreads();
                for (int32_t i = tid; i < count; i += THREADS) {
                    a.dst_cols[out0 + i] = c0 + (int32_t)(o_place[i] >> 8);
                    a.dst_rows[out0 + i] = (int32_t)r0 + (int32_t)(o_place[i] & 255u);
                    a.dst_vals[out0 + i] = o_val[i];
                }
            }
        }
        out0 += entries_of_window;
        if (RANKED) __syncthreads();                         // the masks and the sums are read before the next window's
    }
}

template <int WORDS, OrderKind KIND, int THREADS = kOrderThreads>
__global__ __launch_bounds__(THREADS) void order_groups(OrderArgs a)
{
    order_part<WORDS, KIND, THREADS>(a, (int32_t)blockIdx.x);
}

// A part per group; the input's columns have 16 bits (OrderArgs::cols points to them).
template <int WORDS, int THREADS>
__global__ __launch_bounds__(THREADS) void order_groups_host(OrderArgs a, GroupStarts starts)
{
    order_part<WORDS, kOrderHost, THREADS>(a, (int32_t)blockIdx.x, starts.at[blockIdx.x], starts.at[blockIdx.x + 1]);
}

// order_groups and band_fill in one launch, the lists first: neither needs anything of the other, both wait for LDS and memory most of their time, and neither fills the
// chip by itself.  Six waves per SIMD and four entries per thread and step: with eight entries the registers spill (4000 x 4000, 5 %, whole conversion: 24.0 us,
// 29.7 without the limit, 23.8 so).  Dynamic LDS: the larger of the two.
constexpr int kBothThreads = 512;
template <int WORDS, OrderKind KIND, int V>
__global__ __launch_bounds__(kBothThreads, 6) void order_and_fill(OrderArgs a, FillArgs f, int32_t lists)
{
    if ((int32_t)blockIdx.x < lists) band_fill_list<V, kBothThreads, 4>(f, blockIdx.x);
    else order_part<WORDS, KIND, kBothThreads>(a, (int32_t)blockIdx.x - lists);
}

}  // namespace gcoo
