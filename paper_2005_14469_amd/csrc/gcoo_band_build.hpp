// Kernels that write the band schedule (layout in gcoo_band.hpp) from the entries in row order: band_mark, one bitmap of
// columns per wave list, then band_fill, heads and units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcoo_band.hpp"
#include "gcoo_build_kernels.hpp"

namespace gcoo {

constexpr int kBandMarkThreads = 512;
constexpr int kBandChunk = 14400;                        // distinct columns that band_fill holds at a time, at most (whole bands of both cuts)
constexpr int kBandGroup = 5;                            // columns of a band that one lane counts

// Entries of a list: the rows [list * h, + h) of A.
struct BandList {
    int64_t r0;
    int32_t rows, beg, end;
};
__device__ __forceinline__ BandList band_list(const int32_t* __restrict__ row_start, int64_t m, int32_t h, int64_t list)
{
    BandList l;
    l.r0 = list * h;
    if (l.r0 > m) l.r0 = m;
    l.rows = (int32_t)(m - l.r0 < h ? m - l.r0 : h);
    l.beg = row_start[l.r0];
    l.end = row_start[l.r0 + l.rows];
    return l;
}

// One workgroup per list: parts[list * ceil(k/32) ..] = bitmap of its columns.  Bit sets commute, so the order of the atomics
// is irrelevant.  Dynamic LDS: ceil(k/32) words.
__global__ __launch_bounds__(kBandMarkThreads) void band_mark(const int32_t* __restrict__ row_start, const int32_t* __restrict__ row_cols,
                                                              int64_t m, int64_t k, int32_t h, uint32_t* __restrict__ parts,
                                                              int32_t heavy, uint32_t* __restrict__ uneven)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t band_lds[];
    const int32_t nbw = (int32_t)((k + 31) / 32);
    const BandList l = band_list(row_start, m, h, blockIdx.x);
    if (threadIdx.x == 0 && l.end - l.beg > heavy) *uneven = 1u;      // (zero so far)
    for (int32_t i = threadIdx.x; i < nbw; i += kBandMarkThreads) band_lds[i] = 0u;
    __syncthreads();
    for (int32_t e = l.beg + (int32_t)threadIdx.x; e < l.end; e += 4 * kBandMarkThreads) {
        uint32_t c[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) c[x] = e + x * kBandMarkThreads < l.end ? (uint32_t)row_cols[e + x * kBandMarkThreads] : 0xffffffffu;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            if (e + x * kBandMarkThreads >= l.end) break;
            const uint32_t col = c[x] < (uint32_t)k ? c[x] : (uint32_t)k - 1u;
            atomicOr(&band_lds[col >> 5], 1u << (col & 31u));
        }
    }
    __syncthreads();
    uint32_t* out = parts + (int64_t)blockIdx.x * nbw;
    for (int32_t i = threadIdx.x; i < nbw; i += kBandMarkThreads) out[i] = band_lds[i];
}

// Exclusive prefix sum of x over every stretch of LANES (16 or 32) lanes; the stretch's total in *total.
template <int LANES>
__device__ __forceinline__ int32_t band_row_scan(int32_t x, int32_t* total)
{
    const int32_t incl = lanes_scan<LANES>(x);
    if constexpr (LANES == 32) *total = __shfl(incl, (int)(threadIdx.x & 63u) | 31, 64);
    else *total = __builtin_amdgcn_update_dpp(0, incl, 0x15f, 0xf, 0xf, true);  // row_newbcast:15
    return incl - x;
}

// The rows of a list that have an entry in a column as a bit mask of BandCut::kMaxH bits, and above them the pairs and singles of the columns in
// front of it among its five: at most 12 pairs and one single each (24 in the tall cut).
template <int V> struct BandRowMask {
    typedef uint32_t type;
    static __device__ __forceinline__ uint32_t note(uint32_t both) { return ((both & 0xffffu) * 5u + (both >> 16)) << 24; }
    static __device__ __forceinline__ uint32_t in_front(uint32_t word)
    {
        const uint32_t code = word >> 24, pairs = code * 205u >> 10;           // code / 5 below 256
        return pairs | (code - 5u * pairs) << 16;
    }
};
template <> struct BandRowMask<2> {
    typedef unsigned long long type;
    static __device__ __forceinline__ unsigned long long note(uint32_t both) { return (unsigned long long)((both & 0xffffu) | (both >> 16) << 8) << 48; }
    static __device__ __forceinline__ uint32_t in_front(unsigned long long word)
    {
        const uint32_t code = (uint32_t)(word >> 48);
        return (code & 0xffu) | (code >> 8) << 16;
    }
};
__device__ __forceinline__ uint32_t band_popc(uint32_t x) { return (uint32_t)__popc(x); }
__device__ __forceinline__ uint32_t band_popc(unsigned long long x) { return (uint32_t)__popcll(x); }

// Dynamic LDS of band_fill: the column words of a block, a mask per column of the chunk, a place per five of them.
inline size_t band_fill_lds(int64_t k, int64_t chunk, int v)
{
    return (size_t)((k + 31) / 32) * 8 + (size_t)chunk * (v == 4 ? 4 : 8) + (size_t)(chunk / kBandGroup) * 4;
}

// One workgroup per wave's list.  The columns of the block are the OR of its bitmaps; their popcounts, summed up, give a
// column its place among the distinct ones.  A mask per distinct column collects the rows that hold an entry in it
// (bit sets again, so nothing depends on timing), and from those masks follow, without a sort, the pairs and singles of every
// band and the place of every entry in them.  A coordinate that occurs twice sets its bit twice: such a list is written the
// slow way, a wave per band that picks the band's entries from the whole list in order.
// Every list has a stretch of the units to itself, as long as its entries and bands can make it, so that none waits for the others to be counted.
// Bound: latency up to a few thousand entries per list.  A thread has few of them, and every step is a chain of LDS reads, so what waits for nothing but
// the rows' bounds is asked for first, EACH entries per thread go through a step side by side and are kept for the next (where all of them are), sixteen lanes
// count a band, a column's place in its band is in its mask word and one word per five columns, and a wave finds the rows of its 64 entries from the
// starts in its lanes.  (4000 x 4000, 2 %: 13.6 -> 10.2 us, 5 %: 17.6 -> 12.6; 8000 x 8000, 0.5 %, tall: 15.9 -> 12.2; 14000 x 14000, 2 %: 103 -> 53.)
// Longer lists come to 75 to 80 records per ns, 8 bytes each to a line of its own (8000 x 8000, 10 %: 83 us); putting a stretch of units together in LDS
// and writing it in whole lines took as long (84 to 121 us for 48 to 8 KB), and so did going through the entries once for each half of the columns (88).
// V as in BandCut.  kBandBuildThreads = 1024 for lists of many entries, of which there are too few to fill the chip with workgroups of 512.
// Dynamic LDS: band_fill_lds().
struct FillArgs {
    const int32_t* row_start;
    const int32_t* row_cols;
    const float* row_vals;
    int64_t m, k;
    int32_t h, chunk;
    const uint32_t* parts;
    int64_t head_stride;
    uint32_t* head;
    uint32_t* units;
    int32_t* first;
    int32_t* count;
    const uint32_t* uneven;    // not 0: the product goes row by row; or null and
    const uint32_t* flags;     // the word of every list, in some of which a bit of `heavy` says so
    int32_t flag_count;
    uint32_t heavy;
    RowsOut out;               // GROUPED only
    uint32_t* says_uneven;
    uint32_t* soon;            // the same for this launch, cleared by the one before it, on a line of its own: the count of the long rows lies beside the other
    int64_t g;
    int32_t p;
};
// GROUPED: behind fill_dense_groups().  The bitmaps are those of the groups, and no launch before this one could list the long rows or say that the lists are uneven, `flag_count` lists (as in
// band_mark) of at most `heavy` entries where they are not: this one does, the list of a wave for its own rows, and the lists in front for the matrix (band_tests()).
template <int V, int kBandBuildThreads, int EACH, bool GROUPED = false>
__device__ __forceinline__ void band_fill_list(const FillArgs& a, int64_t list)
{
    typedef BandCut<V> Cut;
    typedef typename BandRowMask<V>::type Mask;
    constexpr int kBandBuildWaves = kBandBuildThreads / 64, kBandRows = Cut::kRows, kBandChunkBands = kBandChunk / kBandRows;
    constexpr int kParts = kBandWaves * 4 / V;             // bitmaps of a block, band_lists_of(V) per wave
    constexpr int kLanes = kBandRows / kBandGroup;       // lanes that count a band
    constexpr int kHeld = EACH * kBandBuildThreads;         // entries that the threads keep from the counts to the records
    constexpr Mask kRowsOnly = ((Mask)1 << Cut::kMaxH) - 1;
    static_assert(kBandChunk % kBandRows == 0 && kBandChunkBands <= kBandBuildThreads && (kLanes == 16 || kLanes == 32), "");
    extern __shared__ __attribute__((aligned(16))) uint32_t band_lds[];
    __shared__ int32_t wsum[kBandBuildWaves], any_s[kBandBuildWaves], repeated_s;
    __shared__ int2 band_s[kBandChunkBands];                // first unit and pairs of a band
    __shared__ int32_t singles_s[kBandChunkBands];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t m = a.m, k = a.k, Q = list / kBandWaves;
    const int32_t h = a.h, chunk = a.chunk, w = (int32_t)(list - Q * kBandWaves);
    const int32_t* __restrict__ row_start = a.row_start;
    const int32_t* __restrict__ row_cols = a.row_cols;
    const float* __restrict__ row_vals = a.row_vals;
    const uint32_t* __restrict__ parts = a.parts;
    const int32_t nbw = (int32_t)((k + 31) / 32);
    uint2* words = (uint2*)band_lds;                        // the block's columns, and the distinct ones in front of a word of them
    Mask* rows_of = (Mask*)(words + nbw);                   // rows of the list with an entry in a column of the chunk
    uint32_t* place_of = (uint32_t*)(rows_of + chunk);      // pairs | singles << 16 of the band in front of five columns
    // What waits for nothing but the rows' bounds is asked for first: the bitmaps, then the entries.
    uint32_t by_rows = 0u, seen = 0u;
    if constexpr (GROUPED) {
        const int64_t each = a.h / band_lists_of(V), from = band_test_from(list, a.flag_count);
        const int32_t tests = band_tests(a.flag_count);
        if (tests < a.flag_count) seen = __hip_atomic_load(a.soon, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int32_t i = tid; i < tests; i += kBandBuildThreads) {
            const int64_t r = (from + i) * each, b = r < m ? r : m, e = b + each < m ? b + each : m;
            by_rows |= (uint32_t)(row_start[e] - row_start[b]) > a.heavy;
        }
    } else if (a.uneven) by_rows = *a.uneven;
    else
        for (int32_t i = tid; i < a.flag_count; i += kBandBuildThreads) by_rows |= a.flags[i] & a.heavy;
    const BandList l = band_list(row_start, m, h, list);
    // word i of the block's columns
    auto columns = [&](int32_t i) {
        uint32_t b = 0u;
        if constexpr (GROUPED) {
            const int64_t r0 = Q * kBandWaves * h, r1 = r0 + kBandWaves * h < m ? r0 + kBandWaves * h : m, q0 = r0 / a.p, q1 = (r1 - 1) / a.p;
            b = parts[(q0 * a.p == r0 ? q0 : a.g + Q) * nbw + i];
            for (int64_t q = q0 + 1; q <= q1; q += 8)
#pragma unroll
                for (int x = 0; x < 8; ++x) b |= parts[(q + x < q1 ? q + x : q1) * nbw + i];      // (the last one again)
        } else {
#pragma unroll
            for (int x = 0; x < kParts; ++x) b |= parts[(Q * kParts + x) * nbw + i];
        }
        return b;
    };
    const uint32_t mine_bits = tid < nbw ? columns(tid) : 0u;
    if (!GROUPED && a.uneven && by_rows != 0u) return;
    const int32_t n = l.end - l.beg, begins = lane < l.rows ? row_start[l.r0 + lane] : INT32_MAX;
    const int32_t* list_cols = row_cols + l.beg;
    const float* list_vals = row_vals + l.beg;
    uint32_t c[EACH];
    float v[EACH];
    auto take = [&](int32_t from) {                         // EACH entries per thread; past the end the first of all again
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            const uint32_t i = (uint32_t)(from + x * kBandBuildThreads + tid), at = i < (uint32_t)n ? i : 0u;
            c[x] = (uint32_t)list_cols[at];
            v[x] = list_vals[at];
        }
    };
    if (n > 0) take(0);
    for (int32_t i = tid; i < chunk; i += kBandBuildThreads) rows_of[i] = 0;
    if (tid < nbw) words[tid].x = mine_bits;
    for (int32_t i = tid + kBandBuildThreads; i < nbw; i += kBandBuildThreads) words[i].x = columns(i);
    if (tid == 0) repeated_s = 0;
    if constexpr (GROUPED) {
        if (wv == 0 && lane < l.rows) list_long_row(a.out, (int32_t)l.r0 + lane, row_start[l.r0 + lane + 1] - begins);
    }
    if (block_any<kBandBuildWaves>((by_rows | seen) != 0u, any_s)) {          // the whole workgroup
        if (GROUPED && __any(by_rows != 0u) && seen == 0u && lane == 0 && band_test_says(list, a.flag_count)) {      // (zero so far)
            *a.says_uneven = 1u;
            __hip_atomic_store(a.soon, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    int32_t nU;
    {
        const int32_t per = (nbw + kBandBuildThreads - 1) / kBandBuildThreads;
        const int32_t i0 = tid * per, i1 = i0 + per < nbw ? i0 + per : nbw;
        int32_t mine = 0;
        for (int32_t i = i0; i < i1; ++i) mine += __popc(words[i].x);
        int32_t at = block_scan<kBandBuildWaves>(mine, wsum, &nU);
        for (int32_t i = i0; i < i1; ++i) {
            words[i].y = (uint32_t)at;
            at += __popc(words[i].x);
        }
    }
    const int32_t NB = (nU + kBandRows - 1) / kBandRows;
    __syncthreads();
    // A list has as many units as its entries and bands can make (band_units()) for itself, so that no list waits for another to be counted.
    const int64_t most = band_max_bands(k, V) * list, base = l.beg / 16 + most + (most < l.beg ? most : l.beg);
    if (tid == 0) {
        a.first[list] = (int32_t)base;
        if (w == 0) a.count[Q] = nU;
    }
    uint32_t* hd = a.head + list * a.head_stride * kBandHeadWords;
    uint2* rec = reinterpret_cast<uint2*>(a.units) + base * 16;

    auto in_range = [&](uint32_t c) -> uint32_t { return c < (uint32_t)k ? c : (uint32_t)k - 1u; };
    auto distinct = [&](uint32_t c) -> int32_t {
        const uint2 x = words[c >> 5];
        return (int32_t)x.y + __popc(x.x & ((1u << (c & 31u)) - 1u));
    };
    // The row of entry e, for all lanes of a wave at once, whose entries ascend from the first lane's on within 64: the rows that begin up to that one, and those that
    // begin behind it.  The lanes hold where the rows begin.
    auto row_of = [&](int32_t e) -> int32_t {
        const int32_t e0 = __builtin_amdgcn_readfirstlane(e);
        int32_t r = __popcll(__ballot(begins <= e0)) - 1;
        for (uint64_t in = __ballot(begins > e0 && begins - e0 < 64); in; in &= in - 1) r += __builtin_amdgcn_readlane(begins, __ffsll((unsigned long long)in) - 1) <= e;
        return r;
    };
    uint32_t key[EACH];                                     // place among the distinct columns << 6 | row
    auto find = [&](int32_t from) {
#pragma unroll
        for (int x = 0; x < EACH; ++x) {
            const int32_t i = from + x * kBandBuildThreads + tid;
            key[x] = (uint32_t)distinct(in_range(c[x])) << 6 | (uint32_t)row_of(l.beg + (i < n ? i : n - 1));
        }
    };

    int32_t listed = 0;                                     // units of the chunks before this one
    for (int32_t u0 = 0; u0 < nU; u0 += chunk) {
        const int32_t nu = u0 + chunk < nU ? chunk : nU - u0, b0 = u0 / kBandRows, bands = (nu + kBandRows - 1) / kBandRows;
        if (u0 > 0) {
            for (int32_t i = tid; i < bands * kBandRows; i += kBandBuildThreads) rows_of[i] = 0;
            __syncthreads();
        }
        for (int32_t from = 0; from < n; from += kHeld) {
            if (from > 0 || (u0 > 0 && n > kHeld)) take(from);
            if (n > kHeld || u0 == 0) find(from);
            Mask old = 0;
#pragma unroll
            for (int x = 0; x < EACH; ++x) {
                const Mask bit = (Mask)1 << (key[x] & 63u);
                const int32_t at = (int32_t)(key[x] >> 6) - u0;
                if (from + x * kBandBuildThreads + tid < n && at >= 0 && at < nu) old |= atomicOr(&rows_of[at], bit) & bit;
            }
            if (old) repeated_s = 1;
        }
        if (u0 == 0) {
            // the columns whose rows the wave fetches, one band beyond the last
            auto column = [&](int32_t i) -> uint32_t {
                i = i < nU ? i : nU - 1;
                int32_t lo = 0, hi = nbw;                   // last word with no more than i in front of it
                while (hi - lo > 1) {
                    const int32_t mid = (lo + hi) >> 1;
                    if ((int32_t)words[mid].y <= i) lo = mid; else hi = mid;
                }
                uint32_t x = words[lo].x;
                for (int32_t j = i - (int32_t)words[lo].y; j > 0; --j) x &= x - 1u;
                return (uint32_t)(lo * 32 + __ffs(x) - 1);
            };
            for (int32_t i = tid; i < (NB + 1) * kBandFetches; i += kBandBuildThreads) {
                const int32_t b = i / kBandFetches, t = i - b * kBandFetches;
                const int32_t first_u = b * kBandRows + (kBandFetches * w + t) * (4 / V);
                uint32_t word = column(first_u);
                if constexpr (V == 2) word |= (column(first_u + 1) - word) << 16;
                hd[b * kBandHeadWords + t] = word;
            }
        }
        __syncthreads();
        const bool repeated = repeated_s != 0;
        if (repeated) {
            for (int32_t b = wv; b < bands; b += kBandBuildWaves) {
                int32_t sum = 0;
                for (int32_t cur = l.beg; cur < l.end; cur += 64) {
                    const int32_t e = cur + lane;
                    sum += __popcll(__ballot(e < l.end && distinct(in_range((uint32_t)row_cols[e < l.end ? e : l.beg])) / kBandRows == b0 + b));
                }
                if (lane == 0) {
                    band_s[b].y = 0;
                    singles_s[b] = sum;
                }
            }
        } else {
            // five columns per lane
            constexpr int kPerWave = 64 / kLanes;
            for (int32_t b = wv * kPerWave; b < bands; b += kBandBuildWaves * kPerWave) {
                const int32_t mine = b + lane / kLanes, at = mine * kBandRows + lane % kLanes * kBandGroup;
                uint32_t both = 0u;
                if (mine < bands) {
#pragma unroll
                    for (int x = 0; x < kBandGroup; ++x) {
                        const Mask rows = rows_of[at + x];
                        if (x > 0) rows_of[at + x] = rows | BandRowMask<V>::note(both);
                        const uint32_t cnt = band_popc(rows);
                        both += (cnt >> 1) | (cnt & 1u) << 16;
                    }
                }
                int32_t total;
                const int32_t in_front = band_row_scan<kLanes>((int32_t)both, &total);
                if (mine < bands) {
                    place_of[at / kBandGroup] = (uint32_t)in_front;
                    if (lane % kLanes == 0) {
                        band_s[mine].y = total & 0xffff;
                        singles_s[mine] = total >> 16;
                    }
                }
            }
        }
        __syncthreads();
        // units in front of every band of the chunk
        int32_t units_here;
        {
            const int32_t ps = tid < bands ? (band_s[tid].y + 1) / 2 : 0, ss = tid < bands ? (singles_s[tid] + 3) / 4 : 0;
            const int32_t mine = tid < bands ? (ps + ss > 0 ? (ps + ss + 3) / 4 : 1) : 0;
            const int32_t off = block_scan<kBandBuildWaves>(mine, wsum, &units_here);
            if (tid < bands) {
                band_s[tid].x = off;
                hd[(b0 + tid + 1) * kBandHeadWords + 5] = (uint32_t)ps;
                hd[(b0 + tid + 1) * kBandHeadWords + 6] = (uint32_t)ss;
            }
        }
        __syncthreads();
        uint2* chunk_rec = rec + (int64_t)listed * 16;
        listed += units_here;
        if (!repeated) {
            for (int32_t from = 0; from < n; from += kHeld) {
                if (n > kHeld) {
                    take(from);
                    find(from);
                }
#pragma unroll
                for (int x = 0; x < EACH; ++x) {
                    const int32_t at = (int32_t)(key[x] >> 6) - u0;
                    if (from + x * kBandBuildThreads + tid >= n || at < 0 || at >= nu) continue;
                    const int32_t r = (int32_t)(key[x] & 63u), b = at / kBandRows;
                    const Mask word = rows_of[at], rows = word & kRowsOnly;
                    const uint32_t front = place_of[at / kBandGroup] + BandRowMask<V>::in_front(word);
                    const int2 band = band_s[b];
                    const int32_t cnt = (int32_t)band_popc(rows), mine = (int32_t)band_popc(rows & (((Mask)1 << r) - 1));
                    const int32_t idx = (mine == cnt - 1 && (cnt & 1)) ? 4 * ((band.y + 1) / 2) + (int32_t)(front >> 16) : 2 * (int32_t)(front & 0xffffu) + mine;
                    chunk_rec[band.x * 16 + idx] = make_uint2(__float_as_uint(v[x]),
                                                              (uint32_t)r | (uint32_t)(((b0 + b) & 1) * kBandRows + at - b * kBandRows) << Cut::kPlaceShift);
                }
            }
        } else {
            for (int32_t b = wv; b < bands; b += kBandBuildWaves) {
                uint2* to = chunk_rec + band_s[b].x * 16;
                int32_t done = 0;
                for (int32_t cur = l.beg; cur < l.end; cur += 64) {
                    const int32_t e = cur + lane;
                    const int32_t at = distinct(in_range((uint32_t)row_cols[e < l.end ? e : l.beg]));
                    const bool mine = e < l.end && at / kBandRows == b0 + b;
                    const int32_t r = row_of(e < l.end ? e : l.end - 1);
                    const uint64_t mk = __ballot(mine);
                    if (mine)
                        to[done + __popcll(mk & ((1ull << lane) - 1ull))] = make_uint2(__float_as_uint(row_vals[e]),
                            (uint32_t)r | (uint32_t)(((b0 + b) & 1) * kBandRows + at - (b0 + b) * kBandRows) << Cut::kPlaceShift);
                    done += __popcll(mk);
                }
            }
        }
        // the records without an entry: at most two behind the pairs, up to a unit behind the singles (sixteen lanes per band)
        for (int32_t b = tid >> 4; b < bands; b += kBandBuildThreads / 16) {
            const int32_t np = band_s[b].y, ns = singles_s[b], ps = (np + 1) / 2, ss = (ns + 3) / 4;
            const int32_t room = 16 * (ps + ss > 0 ? (ps + ss + 3) / 4 : 1), i = tid & 15;
            uint2* to = chunk_rec + band_s[b].x * 16;
            const uint2 none = make_uint2(0u, (uint32_t)Cut::kSink);
            if (2 * np + i < 4 * ps) to[2 * np + i] = none;
            if (4 * ps + ns + i < room) to[4 * ps + ns + i] = none;
        }
        if (u0 + chunk < nU) __syncthreads();
    }
}

template <int V, int kBandBuildThreads, int EACH, bool GROUPED>
__global__ __launch_bounds__(kBandBuildThreads) void band_fill(FillArgs a)
{
    band_fill_list<V, kBandBuildThreads, EACH, GROUPED>(a, blockIdx.x);
}

}  // namespace gcoo
