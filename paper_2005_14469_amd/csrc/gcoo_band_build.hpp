// Kernels that write the band schedule (layout in gcoo_band.hpp) from the entries in row order: band_mark, one bitmap of
// columns per wave list, then band_fill, heads and units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcoo_band.hpp"

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
                                                              uint32_t* __restrict__ zeroed, int32_t heavy, uint32_t* __restrict__ uneven)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t band_lds[];
    if (blockIdx.x == 0 && threadIdx.x == 0) *zeroed = 0u;            // the counter from which band_fill places the lists
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

// Exclusive prefix sum over the workgroup; the total in *total (shared).
template <int kBandBuildThreads>
__device__ __forceinline__ int32_t band_block_scan(int32_t mine, int32_t* wsum, int32_t* total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int32_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int32_t off = incl - mine;
    for (int j = 0; j < wv; ++j) off += wsum[j];
    if (threadIdx.x == kBandBuildThreads - 1) *total = off + mine;
    __syncthreads();
    return off;
}

// Exclusive prefix sum of x over every stretch of LANES (16 or 32) lanes; the stretch's total in *total.
template <int LANES>
__device__ __forceinline__ int32_t band_row_scan(int32_t x, int32_t* total)
{
    int32_t incl = x;
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);
    if constexpr (LANES == 32) {
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);  // row_bcast:15, into rows 1 and 3
        *total = __shfl(incl, (int)(threadIdx.x & 63u) | 31, 64);
    } else {
        *total = __builtin_amdgcn_update_dpp(0, incl, 0x15f, 0xf, 0xf, true);  // row_newbcast:15
    }
    return incl - x;
}

// The rows of a list as a bit mask.
template <int V> struct BandRowMask { typedef uint32_t type; };
template <> struct BandRowMask<2> { typedef unsigned long long type; };
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
// Bound: latency.  A list is a few hundred to a few thousand entries, so a thread has few of them, and every step is a chain of LDS reads: four
// entries per thread go through it side by side, sixteen lanes count a band, four bands per wave, and the LDS per column is kept
// small enough for four workgroups per compute unit (8000 x 8000, 0.5 %: 31 us with a band per wave and two workgroups, 17 us so).
// V as in BandCut.  kBandBuildThreads = 1024 for lists of many entries, of which there are too few to fill the chip with workgroups of 512.
// Dynamic LDS: band_fill_lds().
template <int V, int kBandBuildThreads>
__global__ __launch_bounds__(kBandBuildThreads) void band_fill(const int32_t* __restrict__ row_start, const int32_t* __restrict__ row_cols,
                                                              const float* __restrict__ row_vals, int64_t m, int64_t k, int32_t h,
                                                              const uint32_t* __restrict__ parts, int32_t chunk, int64_t capacity,
                                                              int64_t head_stride, uint32_t* __restrict__ head, uint32_t* __restrict__ units,
                                                              int32_t* __restrict__ first, int32_t* __restrict__ count, uint32_t* __restrict__ alloc,
                                                              const uint32_t* __restrict__ uneven)
{
    if (*uneven != 0u) return;                                 // the product goes row by row
    typedef BandCut<V> Cut;
    typedef typename BandRowMask<V>::type Mask;
    constexpr int kBandBuildWaves = kBandBuildThreads / 64, kBandRows = Cut::kRows, kBandChunkBands = kBandChunk / kBandRows;
    constexpr int kParts = kBandWaves * 4 / V;             // bitmaps of a block, band_lists_of(V) per wave
    constexpr int kFind = V == 4 ? 32 : 64, kLanes = kBandRows / kBandGroup;       // lanes that count a band
    static_assert(kBandChunk % kBandRows == 0 && kBandChunkBands <= kBandBuildThreads && Cut::kMaxH < kFind && (kLanes == 16 || kLanes == 32), "");
    extern __shared__ __attribute__((aligned(16))) uint32_t band_lds[];
    __shared__ int32_t wsum[kBandBuildWaves], total_s, repeated_s, base_s, rs[kFind];
    __shared__ int32_t pairs_s[kBandChunkBands], singles_s[kBandChunkBands], at_s[kBandChunkBands];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t nbw = (int32_t)((k + 31) / 32);
    uint32_t* bits = band_lds;                              // the block's columns
    int32_t* before = (int32_t*)(bits + nbw);               // distinct columns in front of a word of them
    Mask* rows_of = (Mask*)(before + nbw);                  // rows of the list with an entry in a column of the chunk
    uint32_t* place_of = (uint32_t*)(rows_of + chunk);      // pairs | singles << 16 of the band in front of five columns
    const int64_t list = blockIdx.x, Q = list / kBandWaves;
    const int32_t w = (int32_t)(list - Q * kBandWaves);
    const BandList l = band_list(row_start, m, h, list);

    for (int32_t i = tid; i < nbw; i += kBandBuildThreads) {
        uint32_t b = 0u;
#pragma unroll
        for (int x = 0; x < kParts; ++x) b |= parts[(Q * kParts + x) * nbw + i];
        bits[i] = b;
    }
    // where the rows begin; places past the last row hold a number no entry reaches, so that the search below always takes as many steps
    if (tid < kFind) rs[tid] = tid <= l.rows ? row_start[l.r0 + tid] : INT32_MAX;
    if (tid == 0) repeated_s = 0;
    __syncthreads();
    if (tid == 0) rs[l.rows] = INT32_MAX;
    {
        const int32_t per = (nbw + kBandBuildThreads - 1) / kBandBuildThreads;
        const int32_t i0 = tid * per, i1 = i0 + per < nbw ? i0 + per : nbw;
        int32_t mine = 0;
        for (int32_t i = i0; i < i1; ++i) mine += __popc(bits[i]);
        int32_t at = band_block_scan<kBandBuildThreads>(mine, wsum, &total_s);
        for (int32_t i = i0; i < i1; ++i) {
            before[i] = at;
            at += __popc(bits[i]);
        }
    }
    const int32_t nU = total_s, NB = (nU + kBandRows - 1) / kBandRows;
    __syncthreads();
    if (tid == 0 && w == 0) count[Q] = nU;
    uint32_t* hd = head + list * head_stride * kBandHeadWords;
    // the columns whose rows the wave fetches, one band beyond the last
    auto column = [&](int32_t u) -> uint32_t {
        u = u < nU ? u : nU - 1;
        int32_t lo = 0, hi = nbw;                           // last word with before[] <= u
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (before[mid] <= u) lo = mid; else hi = mid;
        }
        uint32_t x = bits[lo];
        for (int32_t n = u - before[lo]; n > 0; --n) x &= x - 1u;
        return (uint32_t)(lo * 32 + __ffs(x) - 1);
    };
    for (int32_t i = tid; i < (NB + 1) * kBandFetches && nU > 0; i += kBandBuildThreads) {
        const int32_t b = i / kBandFetches, t = i - b * kBandFetches;
        const int32_t u = b * kBandRows + (kBandFetches * w + t) * (4 / V);
        uint32_t c = column(u);
        if constexpr (V == 2) c |= (column(u + 1) - c) << 16;
        hd[b * kBandHeadWords + t] = c;
    }

    auto in_range = [&](uint32_t c) -> uint32_t { return c < (uint32_t)k ? c : (uint32_t)k - 1u; };
    auto distinct = [&](uint32_t c) -> int32_t { return before[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31u)) - 1u)); };
    auto row_of = [&](int32_t e) -> int32_t {
        int32_t r = 0;
#pragma unroll
        for (int d = kFind / 2; d >= 1; d >>= 1) r += rs[r + d] <= e ? d : 0;
        return r;
    };

    // Two rounds over the chunks of distinct columns: the first counts the units, the second writes; with one chunk what the
    // first round found is still there.
    const int32_t chunks = (nU + chunk - 1) / chunk;
    int32_t listed = 0;                                     // units of the chunks before this one
    for (int round = 0; round < 2; ++round) {
        listed = 0;
        for (int32_t ch = 0; ch < chunks; ++ch) {
            const int32_t u0 = ch * chunk, nu = u0 + chunk < nU ? chunk : nU - u0, b0 = u0 / kBandRows, bands = (nu + kBandRows - 1) / kBandRows;
            if (round == 0 || chunks > 1) {
                for (int32_t i = tid; i < bands * kBandRows; i += kBandBuildThreads) rows_of[i] = 0;
                __syncthreads();
                for (int32_t e = l.beg + tid; e < l.end; e += 4 * kBandBuildThreads) {
                    uint32_t c[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int32_t at = e + x * kBandBuildThreads;
                        c[x] = (uint32_t)row_cols[at < l.end ? at : e];
                    }
                    int32_t u[4];
                    Mask bit[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        u[x] = distinct(in_range(c[x])) - u0;
                        bit[x] = (Mask)1 << row_of(e + x * kBandBuildThreads);
                    }
                    Mask old[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        old[x] = 0;
                        if (e + x * kBandBuildThreads < l.end && u[x] >= 0 && u[x] < nu) old[x] = atomicOr(&rows_of[u[x]], bit[x]) & bit[x];
                    }
                    if (old[0] | old[1] | old[2] | old[3]) repeated_s = 1;
                }
                __syncthreads();
                const bool repeated = repeated_s != 0;
                if (repeated) {
                    for (int32_t b = wv; b < bands; b += kBandBuildWaves) {
                        int32_t n = 0;
                        for (int32_t cur = l.beg; cur < l.end; cur += 64) {
                            const int32_t e = cur + lane;
                            n += __popcll(__ballot(e < l.end && distinct(in_range((uint32_t)row_cols[e < l.end ? e : l.beg])) / kBandRows == b0 + b));
                        }
                        if (lane == 0) {
                            pairs_s[b] = 0;
                            singles_s[b] = n;
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
                                const uint32_t n = band_popc(rows_of[at + x]);
                                both += (n >> 1) | (n & 1u) << 16;
                            }
                        }
                        int32_t total;
                        const int32_t in_front = band_row_scan<kLanes>((int32_t)both, &total);
                        if (mine < bands) {
                            place_of[at / kBandGroup] = (uint32_t)in_front;
                            if (lane % kLanes == 0) {
                                pairs_s[mine] = total & 0xffff;
                                singles_s[mine] = total >> 16;
                            }
                        }
                    }
                }
                __syncthreads();
                // units in front of every band of the chunk
                const int32_t steps = tid < bands ? (pairs_s[tid] + 1) / 2 + (singles_s[tid] + 3) / 4 : 0;
                const int32_t mine = tid < bands ? (steps > 0 ? (steps + 3) / 4 : 1) : 0;
                const int32_t off = band_block_scan<kBandBuildThreads>(mine, wsum, &total_s);
                if (tid < bands) at_s[tid] = listed + off;
                listed += total_s;
                __syncthreads();
            }
            if (round == 0) continue;
            // a list that does not fit (only with offsets of rows that contradict each other) is left empty
            const bool fits = base_s >= 0;
            if (tid < bands) {
                hd[(b0 + tid + 1) * kBandHeadWords + 5] = fits ? (uint32_t)((pairs_s[tid] + 1) / 2) : 0u;
                hd[(b0 + tid + 1) * kBandHeadWords + 6] = fits ? (uint32_t)((singles_s[tid] + 3) / 4) : 0u;
            }
            if (!fits) continue;
            const bool repeated = repeated_s != 0;
            uint2* rec = reinterpret_cast<uint2*>(units) + (int64_t)base_s * 16;
            if (!repeated) {
                for (int32_t e = l.beg + tid; e < l.end; e += 4 * kBandBuildThreads) {
                    uint32_t c[4];
                    float v[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int32_t at = e + x * kBandBuildThreads;
                        c[x] = (uint32_t)row_cols[at < l.end ? at : e];
                        v[x] = row_vals[at < l.end ? at : e];
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int32_t u = distinct(in_range(c[x])) - u0, row = row_of(e + x * kBandBuildThreads);
                        if (e + x * kBandBuildThreads >= l.end || u < 0 || u >= nu) continue;
                        const int32_t b = u / kBandRows, g = u / kBandGroup;
                        uint32_t front = place_of[g];
#pragma unroll
                        for (int y = 0; y < kBandGroup - 1; ++y) {
                            const uint32_t n = band_popc(rows_of[g * kBandGroup + y]);
                            front += g * kBandGroup + y < u ? (n >> 1) | (n & 1u) << 16 : 0u;
                        }
                        const Mask rows = rows_of[u];
                        const int32_t n = (int32_t)band_popc(rows), mine = (int32_t)band_popc(rows & (((Mask)1 << row) - 1));
                        const int32_t idx = (mine == n - 1 && (n & 1)) ? 4 * ((pairs_s[b] + 1) / 2) + (int32_t)(front >> 16)
                                                                      : 2 * (int32_t)(front & 0xffffu) + mine;
                        rec[(int64_t)at_s[b] * 16 + idx] = make_uint2(__float_as_uint(v[x]),
                                                                      (uint32_t)row | (uint32_t)(((b0 + b) & 1) * kBandRows + u - b * kBandRows) << Cut::kPlaceShift);
                    }
                }
            } else {
                for (int32_t b = wv; b < bands; b += kBandBuildWaves) {
                    uint2* to = rec + (int64_t)at_s[b] * 16;
                    int32_t done = 0;
                    for (int32_t cur = l.beg; cur < l.end; cur += 64) {
                        const int32_t e = cur + lane;
                        const int32_t u = distinct(in_range((uint32_t)row_cols[e < l.end ? e : l.beg]));
                        const bool mine = e < l.end && u / kBandRows == b0 + b;
                        const uint64_t mk = __ballot(mine);
                        if (mine)
                            to[done + __popcll(mk & ((1ull << lane) - 1ull))] = make_uint2(__float_as_uint(row_vals[e]),
                                (uint32_t)row_of(e) | (uint32_t)(((b0 + b) & 1) * kBandRows + u - (b0 + b) * kBandRows) << Cut::kPlaceShift);
                        done += __popcll(mk);
                    }
                }
            }
            // the records without an entry: at most two behind the pairs, up to a unit behind the singles (sixteen lanes per band)
            for (int32_t b = tid >> 4; b < bands; b += kBandBuildThreads / 16) {
                const int32_t np = pairs_s[b], ns = singles_s[b], ps = (np + 1) / 2, ss = (ns + 3) / 4;
                const int32_t room = 16 * (ps + ss > 0 ? (ps + ss + 3) / 4 : 1), i = tid & 15;
                uint2* to = rec + (int64_t)at_s[b] * 16;
                const uint2 none = make_uint2(0u, (uint32_t)Cut::kSink);
                if (2 * np + i < 4 * ps) to[2 * np + i] = none;
                if (4 * ps + ns + i < room) to[4 * ps + ns + i] = none;
            }
            __syncthreads();
        }
        if (round == 0) {
            if (tid == 0) {
                const int64_t at = atomicAdd(alloc, (uint32_t)listed);
                base_s = at + listed + kBandSlackUnits <= capacity ? (int32_t)at : -1;
                first[list] = base_s < 0 ? 0 : base_s;
            }
            __syncthreads();
        }
    }
}

}  // namespace gcoo
