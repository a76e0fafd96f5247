// SpDM kernel that works row by row: C(r, :) = sum over the stored entries of row r of value x B(column, :).
//
// Where a group has few entries per column (Section 4.1: the mean run is p(1-s)/(1-s^p)), the reuse of a fetched
// value of B that Algorithm 2 is built around finds next to nothing to reuse, and a wave per (group, 256 columns) leaves
// small and narrow products with a handful of waves.  This kernel reads the entries in row order (the copy of them that
// the conversion keeps, gcoo_api.hip), so a partial sum never changes its register, and cuts the work much finer:
//
//   slot      LPR lanes x 4 adjacent columns (LPR = 16, 32 or 64: 64 to 256 columns; 8 and 4 for a narrow B of many rows), one row of A at a time:
//             a wave holds 64 / LPR slots, which load B rows of their own with one instruction
//   entries   16 of a row at a time: every lane loads one (column, value) pair, and a DPP broadcast inside the
//             instruction that uses them hands pair i to the whole slot, so an entry costs one address
//             add, one load and four multiply-adds for 4 x 64 columns at LPR = 16
//   ends      entries past the end of a row have an offset beyond the buffer descriptor's range: the load returns zero
//             without touching memory, so a non-finite B row that no entry touches stays out of C
//   long rows rows of more than `wave_row` entries, and of three times what the rows beside them have, are shared by the slots of the
//             wave: equal stretches, partial sums added in a fixed order, so the bits are the same on every run.  Rows of more
//             than rows_long() are shared by a workgroup and come first: the conversion lists them, and the workgroups of a column
//             tile take one each before their own rows, so that none of them starts when the others have ended
//             (power-law rows, 16384 x 16384, 50 entries on average, N = 512: 100 us; with those of its own rows last 112)
//
// Bound, by the counters: 4 x nnz x N bytes have to come from L2 through the vector caches, which take 64 bytes per clock and compute unit (39 TB/s) at
// the most.  Where the tile of B that an XCD works on stays in its L2 the kernel gets 17 to 23 TB/s of that: 22.7 at 1777 x 2301, 3 %, N = 1117
// (94 % of the requests hit; the tile kernel is faster there), 16.6 to 17.4 at 12000 x 12000, 0.5 %, N = 64.  Where it does not, what the L2 has to fetch counts as well: power-law rows,
// 16384 x 16384, N = 512, whose tile of 64 columns is all of an XCD's 4 MB, take 0.31 GB from behind the L2 for a B of 34 MB (17.8 TB/s from L2);
// 12001 x 12001 with 6 entries per row 2.4 GB for a B of 0.58 GB, which with C is 7.0 TB/s between the L2s and memory where a large copy reaches 5.2:
// there the bound lies behind the L2.  Tiles of 64 columns that fetch 0.76 GB for the aligned rows of 12000 x 12000 take as long as those of 128 that fetch 1.5 (369 and 365 us): memory gives stretches of 256 bytes more slowly.
// Measured (product alone, before = the register kernel): 12000 x 12000, 0.5 %, N = 64: 83 -> 11.0 us; 2500 x 2500, 1 %, N = 1024: 38 -> 15.2; 256 x 256, 10 %, N = 256: 35 -> 4.1;
// 400 x 400, 2 %: 3.4; 4000 x 4000, 2 %, N = 4000: 25 TB/s through the vector cache.  12001 x 12001 as above: 437 us with sixteen rows of B in flight, 427 with eight.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcoo_spdm_launch.hpp"

namespace gcoo {

constexpr int kRowsThreads = 256, kRowsWaves = kRowsThreads / 64;
typedef float rows_f32x4 __attribute__((ext_vector_type(4)));
typedef float rows_f32x4_any __attribute__((ext_vector_type(4), aligned(4)));    // in C, whose rows are aligned to 4 bytes only where the tiles are not moved
typedef uint32_t rows_u32x4 __attribute__((ext_vector_type(4)));

// Pair i of a batch of 16, in every lane of the slot.  LPR >= 16: lane i of every row of 16 lanes holds pair i; below,
// every quad of lanes holds all pairs, pair i in register i / 4 of lane i % 4.
template <int LPR, int I>
__device__ __forceinline__ uint32_t rows_bcast(const uint32_t (&x)[LPR >= 16 ? 1 : 4])
{
    if constexpr (LPR >= 16)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[0], 0x150 + I, 0xf, 0xf, true);                 // row_newbcast:I
    else
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[I / 4], (I % 4) * 0x55, 0xf, 0xf, true);       // quad_perm:[i,i,i,i]
}

// The sum of a row in a lane's four columns, in SUMS parts.
template <int SUMS>
struct RowsAcc {
    float x[SUMS][4] = {};
    __device__ __forceinline__ float total(int u) const
    {
        static_assert(SUMS == 1 || SUMS == 2, "");
        if constexpr (SUMS == 2) return x[0][u] + x[1][u];
        else return x[0][u];
    }
};

// The offset of an entry past the end of its row: no descriptor reaches that far, and a lane's place in the tile (below 2 KB) added to it
// stays below 2^32.  Whoever launches rows_item without WIDE keeps B below kRowsMaxBytes.
constexpr uint32_t kRowsNowhere = 0xfffff000u;
static_assert(kRowsMaxBytes <= kRowsNowhere, "an entry past the end of a row would load an element of B");

// WIDE (a B of more than 4 GB): `off` holds columns, 0xffffffff past the end, and the address is formed in 64 bits.
struct RowsB {
    __amdgpu_buffer_rsrc_t rsrc;
    const char* base;          // WIDE: B, at the descriptor's place
    uint64_t pitch;            // WIDE: bytes
};
// Pairs FROM .. FROM + CNT - 1 of the batch.
template <int LPR, int FROM, int CNT, int I, bool WIDE>
__device__ __forceinline__ void rows_load(const uint32_t (&off)[LPR >= 16 ? 1 : 4], uint32_t lane_off, const RowsB& B, rows_u32x4 (&b)[CNT])
{
    if constexpr (I < CNT) {
        if constexpr (WIDE) {
            const uint32_t col = rows_bcast<LPR, FROM + I>(off);
            b[I] = 0u;
            if (col != 0xffffffffu) __builtin_memcpy(&b[I], B.base + (uint64_t)col * B.pitch + lane_off, 16);
        } else
        b[I] = __builtin_amdgcn_raw_buffer_load_b128(B.rsrc, (int)(rows_bcast<LPR, FROM + I>(off) + lane_off), 0, 0);
        rows_load<LPR, FROM, CNT, I + 1, WIDE>(off, lane_off, B, b);
    }
}
// Adds the pairs of a batch to the sums.  A slot that takes a row by itself which SUMS narrower slots would share is as exact as they are: it keeps SUMS sums, each of every SUMS-th entry
// (KEPT == SUMS), or, where it has not the registers, adds up eight entries by themselves first (KEPT == 1).  Error against 64 bits, 2-norm, by the narrower slots, by one chain in the wider one, and so:
// 333 x 333, rows of 55, N = 333: 1.01e-7 1.36e-7 0.77e-7; 3706 x 5734, rows of 96, N = 27: 0.81e-7 0.99e-7 0.80e-7; power-law rows, 10992 x 10992, N = 85: 1.94e-7 2.62e-7 1.86e-7; 16283 x 16283,
// N = 147: 1.92e-7 3.60e-7 1.46e-7.  Time: level over 110 products of uniform rows, 0.1 % more over 40 of power-law rows, N = 64 to 208 (0.8 % by eights also at 32 lanes; four sums at 64 lanes instead
// of eights: 276 x 276, rows of 22, N = 186: 3.7 4.7 us; 14160 x 14160, rows of 122, N = 134: 74 112).
template <int LPR, int FROM, int CNT, int I, int SUMS, int KEPT>
__device__ __forceinline__ void rows_fma(const uint32_t (&val)[LPR >= 16 ? 1 : 4], const rows_u32x4 (&b)[CNT], float (&part)[4], RowsAcc<KEPT>& acc)
{
    if constexpr (I < CNT) {
        constexpr bool EIGHTS = KEPT != SUMS;
        static_assert(!EIGHTS || KEPT == 1, "");
        const float v = __uint_as_float(rows_bcast<LPR, FROM + I>(val));
        float(&to)[4] = EIGHTS ? part : acc.x[(FROM + I) % KEPT];
#pragma unroll
        for (int u = 0; u < 4; ++u) to[u] = EIGHTS && I % 8 == 0 ? v * __uint_as_float(b[I][u]) : __builtin_fmaf(v, __uint_as_float(b[I][u]), to[u]);
        if constexpr (EIGHTS && (I % 8 == 7 || I == CNT - 1))
#pragma unroll
            for (int u = 0; u < 4; ++u) acc.x[0][u] += part[u];
        rows_fma<LPR, FROM, CNT, I + 1, SUMS>(val, b, part, acc);
    }
}
template <int LPR, int FROM, int CNT, bool WIDE, int SUMS, int KEPT>
__device__ __forceinline__ void rows_batch(const uint32_t (&off)[LPR >= 16 ? 1 : 4], const uint32_t (&val)[LPR >= 16 ? 1 : 4],
                                           uint32_t lane_off, const RowsB& B, RowsAcc<KEPT>& acc)
{
    rows_u32x4 b[CNT];
    rows_load<LPR, FROM, CNT, 0, WIDE>(off, lane_off, B, b);
    float part[4];
    rows_fma<LPR, FROM, CNT, 0, SUMS>(val, b, part, acc);
}

// One (column, value) pair per lane (and register) of a batch of 16 entries: columns beyond the last row of B are brought inside (a
// device CSR input is not checked), entries past `end` get an offset outside the descriptor.
template <int LPR>
struct RowsBatch {
    static constexpr int REGS = LPR >= 16 ? 1 : 4;
    uint32_t c[REGS], v[REGS];
    __device__ __forceinline__ void request(const RowsArgs& a, int32_t base, int32_t end, int lane)
    {
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            const int32_t e = base + (LPR >= 16 ? (lane & 15) : 4 * j + (lane & 3));
            c[j] = 0xffffffffu;
            v[j] = 0u;
            if (e < end) {
                c[j] = (uint32_t)a.cols[e];
                v[j] = __float_as_uint(a.vals[e]);
            }
        }
    }
    template <bool WIDE>
    __device__ __forceinline__ void offsets(uint32_t kmax, uint32_t ldb4)
    {
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            const bool none = c[j] == 0xffffffffu;
            c[j] = c[j] < kmax ? c[j] : kmax;
            if constexpr (WIDE) c[j] = none ? 0xffffffffu : c[j];
            else c[j] = none ? kRowsNowhere : c[j] * ldb4;
        }
    }
};

// The entries from FROM on of the batch, CNT at the most, in steps of two: as many as the fullest slot of the wave has (a load past a row's end returns at once but
// holds the address path as long as any other).
template <int LPR, int FROM, int CNT, bool WIDE, int SUMS, int KEPT>
__device__ __forceinline__ void rows_pick(int32_t left, const RowsBatch<LPR>& now, uint32_t lane_off, const RowsB& B, RowsAcc<KEPT>& acc)
{
    if (__any(left > FROM + CNT - 2)) {
        rows_batch<LPR, FROM, CNT, WIDE, SUMS>(now.c, now.v, lane_off, B, acc);
    } else {
        if constexpr (CNT > 2) rows_pick<LPR, FROM, CNT - 2, WIDE, SUMS>(left, now, lane_off, B, acc);
    }
}

// Adds the entries [base, end) of the slot's row (every lane of the wave calls it; the slots may have different ranges).
// `next` holds the first batch already; on return it holds the batch [more, more_end), requested in front of the loads of
// the last batch.
template <int LPR, bool WIDE, int AHEAD, int SUMS, int KEPT>
__device__ __forceinline__ void rows_entries(const RowsArgs& a, RowsBatch<LPR>& next, int32_t base, int32_t end, int32_t more, int32_t more_end,
                                             uint32_t kmax, uint32_t ldb4, uint32_t lane_off, const RowsB& B, int lane, RowsAcc<KEPT>& acc)
{
    while (true) {
        RowsBatch<LPR> now = next;
        now.template offsets<WIDE>(kmax, ldb4);
        const int32_t left = end - base;
        base += 16;
        const bool last = !__any(base < end);
        next.request(a, last ? more : base, last ? more_end : end, lane);
        rows_pick<LPR, 0, AHEAD, WIDE, SUMS>(left, now, lane_off, B, acc);
        if constexpr (AHEAD < 16)
            if (__any(left > AHEAD)) rows_pick<LPR, AHEAD, 16 - AHEAD, WIDE, SUMS>(left, now, lane_off, B, acc);
        if (last) return;
    }
}

// What a lane needs of a tile of 4 x LPR columns.  AHEAD: loads of rows of B in flight.
template <int LPR, bool WIDE, int AHEAD, int SUMS>
struct RowsTile {
    typedef RowsAcc<AHEAD == 16 && LPR <= 32 ? SUMS : 1> Acc;
    const RowsArgs& a;
    int lane, slot, sl;
    int32_t N, jb, lane_j;
    uint32_t kmax, ldb4, c_word, ldc_word;
    RowsB B;
    __device__ __forceinline__ RowsTile(const RowsArgs& args, int32_t tile) : a(args)
    {
        lane = threadIdx.x & 63;
        slot = lane / LPR;
        sl = lane % LPR;
        const int64_t j0 = (int64_t)tile * (LPR * 4);                 // first column of the tile, less up to `moved` (place())
        // The descriptor starts at or before the first column any lane of the tile loads.
        const int64_t first = j0 - a.moved < 0 ? 0 : (j0 - a.moved < a.N - 4 ? j0 - a.moved : a.N - 4);
        const char* bbase = reinterpret_cast<const char*>(a.B + first);
        const uint64_t bytes = ((uint64_t)(a.k - 1) * (uint64_t)a.ldb + (uint64_t)a.N - (uint64_t)first) * 4u;
        B.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(bbase), 0, (int)(uint32_t)bytes, 0x00027000);
        B.base = bbase;
        B.pitch = (uint64_t)a.ldb * 4u;
        jb = (int32_t)first;
        N = (int32_t)a.N;
        lane_j = (int32_t)j0 + sl * 4;
        ldb4 = (uint32_t)a.ldb * 4u;
        kmax = (uint32_t)(a.k - 1);
        c_word = (uint32_t)(reinterpret_cast<uintptr_t>(a.C) >> 2);
        ldc_word = (uint32_t)a.ldc;
    }
    // A lane's columns in row r: where `moved` is 31 the tile is moved down by what the row's start in C lies past a 128-byte line, so that the
    // stores of a slot are whole lines whatever N and ldc are.  A lane that would reach outside [0, N) loads four columns
    // inside instead and stores those that are its own.
    struct Place { int32_t jc, first, last; };              // elements [first, last) of the vector at column jc
    __device__ __forceinline__ Place place(int32_t r) const
    {
        const int32_t want = lane_j - (int32_t)((c_word + (uint32_t)r * ldc_word) & (uint32_t)a.moved);
        Place pl;
        pl.jc = want < 0 ? 0 : (want > N - 4 ? N - 4 : want);
        pl.first = want - pl.jc < 0 ? 0 : want - pl.jc;
        pl.last = want - pl.jc + 4;
        return pl;
    }
    template <int KEPT>
    __device__ __forceinline__ void store(int32_t r, const Place& pl, const RowsAcc<KEPT>& acc) const
    {
        float* dst = a.C + (int64_t)r * a.ldc + pl.jc;
        if (pl.first == 0 && pl.last >= 4) {
            rows_f32x4 o = {acc.total(0), acc.total(1), acc.total(2), acc.total(3)};
            __builtin_nontemporal_store(o, reinterpret_cast<rows_f32x4_any*>(dst));
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u >= pl.first && u < pl.last) __builtin_nontemporal_store(acc.total(u), dst + u);
        }
    }
    __device__ __forceinline__ void entries(RowsBatch<LPR>& next, int32_t base, int32_t end, int32_t more, int32_t more_end, const Place& pl, Acc& acc) const
    {
        rows_entries<LPR, WIDE, AHEAD, SUMS>(a, next, base, end, more, more_end, kmax, ldb4, (uint32_t)(pl.jc - jb) * 4u, B, lane, acc);
    }
    // The entries [b, e) of row r, equal stretches of them for the slots of the wave; the sums of the slots added up in a fixed tree.
    __device__ __forceinline__ RowsAcc<1> shared_row(const Place& pl, int32_t b, int32_t e) const
    {
        RowsBatch<LPR> mine;
        mine.request(a, b, e, lane);
        Acc all;
        entries(mine, b, e, 0, 0, pl, all);
        RowsAcc<1> sum;
#pragma unroll
        for (int u = 0; u < 4; ++u) sum.x[0][u] = all.total(u);
#pragma unroll
        for (int d = LPR; d < 64; d <<= 1)
#pragma unroll
            for (int u = 0; u < 4; ++u) sum.x[0][u] += __shfl_xor(sum.x[0][u], d, 64);
        return sum;
    }
};

// Where the long rows are: in a list, or in places, which workgroups begin with in their order or by rows_turn().
enum RowsLong { kLongCounted, kLongPlaces, kLongSpread };

// The long rows `turn`, `turn` + step, ..., the `n_front` longest first, all slots of a workgroup on each.  `part`: a stretch of a tile's columns per wave in LDS.  PLACES: the long rows are
// in places, not counted (RowsArgs), and place `turn` holds `at_turn`.
template <int LPR, bool WIDE, int AHEAD, int SUMS, RowsLong LONG>
__device__ __forceinline__ void rows_long_rows(const RowsTile<LPR, WIDE, AHEAD, SUMS>& T, int32_t n_front, int32_t n_long, int32_t turn, int32_t step, int32_t at_turn, float (*part)[LPR * 4])
{
    constexpr bool PLACES = LONG != kLongCounted;
    constexpr int SPW = 64 / LPR, SLOTS = SPW * kRowsWaves;
    const RowsArgs& a = T.a;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int32_t x = turn; x < n_long; x += step) {
        const int32_t lr = __builtin_amdgcn_readfirstlane(PLACES ? (x == turn ? at_turn : a.long_rows[x]) : a.long_rows[x < n_front ? x : a.long_room - 1 - (x - n_front)]);
        if (PLACES && (lr < 0 || lr >= (int32_t)a.m)) continue;                      // a place without a row
        const int32_t lb = a.row_ptr[lr], le = a.row_ptr[lr + 1];
        if (PLACES && le - lb <= a.long_row) continue;
        const int32_t each = (le - lb + SLOTS - 1) / SLOTS, b = lb + (wv * SPW + T.slot) * each, e = b + each < le ? b + each : le;
        const typename RowsTile<LPR, WIDE, AHEAD, SUMS>::Place lpl = T.place(lr);
        RowsAcc<1> sum = T.shared_row(lpl, b, e);
        if (T.slot == 0)
#pragma unroll
            for (int u = 0; u < 4; ++u) part[wv][T.sl * 4 + u] = sum.x[0][u];
        __syncthreads();
        if (wv == 0 && T.slot == 0) {
            for (int s = 1; s < kRowsWaves; ++s)
#pragma unroll
                for (int u = 0; u < 4; ++u) sum.x[0][u] += part[s][T.sl * 4 + u];
            T.store(lr, lpl, sum);
        }
        __syncthreads();
    }
}

// The wave's rows [w0, w0 + wrows), a slot on each; lane i holds in `start` where row w0 + i begins, i = 0 .. wrows.  Rows of more than `long_row` entries, which is no less
// than `wave_row`, are left out.
template <int LPR, bool WIDE, int AHEAD, int SUMS>
__device__ __forceinline__ void rows_of_wave(const RowsTile<LPR, WIDE, AHEAD, SUMS>& T, int32_t w0, int32_t wrows, int32_t start, int32_t wave_row, int32_t long_row)
{
    constexpr int SPW = 64 / LPR;
    const RowsArgs& a = T.a;
    auto bounds = [&](int32_t i, int32_t* beg, int32_t* end) {                      // of the wave's row i (empty past the last)
        const int32_t b = __shfl(start, i, 64), e = __shfl(start, i + 1, 64);
        *beg = b;
        *end = i < wrows ? e : b;
    };
    int32_t beg, end;
    bounds(T.slot, &beg, &end);
    // the row is left to all slots of the wave (or, when it is a long one, to nobody here)
    auto shared = [&](int32_t n) {
        if (!__any(n > 16)) return n > wave_row;
        int32_t all = n;
#pragma unroll
        for (int d = LPR; d < 64; d <<= 1) all += __shfl_xor(all, d, 64);
        return n > wave_row || (n > 16 && n * (SPW - 1) > 3 * (all - n));
    };
    RowsBatch<LPR> next;
    bool whole = shared(end - beg);
    next.request(a, beg, whole ? beg : end, T.lane);
    for (int32_t i = 0; i < wrows; i += SPW) {
        const int32_t r = w0 + i + T.slot;
        int32_t beg2, end2;
        bounds(i + SPW + T.slot, &beg2, &end2);
        const bool whole2 = shared(end2 - beg2);
        const typename RowsTile<LPR, WIDE, AHEAD, SUMS>::Place pl = T.place(r);
        typename RowsTile<LPR, WIDE, AHEAD, SUMS>::Acc acc;
        T.entries(next, beg, whole ? beg : end, beg2, whole2 ? beg2 : end2, pl, acc);
        if (i + T.slot < wrows && !whole) T.store(r, pl, acc);
        uint64_t todo = __ballot(whole && T.sl == 0);
        while (todo) {                                                              // wave-uniform
            const int32_t s = (__ffsll((long long)todo) - 1) / LPR;
            todo &= todo - 1;
            const int32_t lb = __builtin_amdgcn_readlane(start, i + s), le = __builtin_amdgcn_readlane(start, i + s + 1);
            const int32_t lr = w0 + i + s, n = le - lb;
            if (n > long_row) continue;
            const int32_t each = (n + SPW - 1) / SPW, b = lb + T.slot * each, e = b + each < le ? b + each : le;
            const typename RowsTile<LPR, WIDE, AHEAD, SUMS>::Place lpl = T.place(lr);
            const RowsAcc<1> sum = T.shared_row(lpl, b, e);
            if (T.slot == 0) T.store(lr, lpl, sum);
        }
        beg = beg2;
        end = end2;
        whole = whole2;
    }
}

// Item `block`, (tile, wg): rows [wg * kRowsWaves * rpw, ...), `rpw` of them per wave, columns of the tile.  Where the long rows are is a template, since the
// places in the one kernel cost the other matrices up to 3 % (12000 x 12000, 0.5 %, N = 64: 12.08 and 12.20 us).
template <int LPR, bool WIDE, int AHEAD, int SUMS, RowsLong LONG>
__device__ __forceinline__ void rows_item(const RowsArgs& a, uint32_t block, int32_t tiles, int32_t row_wgs, int32_t rpw, int32_t wave_row, const RowsTurns& turns, float (*part)[LPR * 4])
{
    // XCD-aware order: an XCD walks all rows of one column tile before the next, so that the tile of B stays in its L2, and the
    // eight XCDs work on eight tiles side by side, so that what they read and write of a row at about the same time is one
    // stretch of 2 KB.  The tiles beyond the last whole eight are cut into eight slices of rows.
    constexpr bool PLACES = LONG != kLongCounted;
    const int32_t xcd = (int32_t)(block & 7u), at = (int32_t)(block >> 3), eights = tiles / 8;
    int32_t tile, wg, slice = 0;                                     // slice: workgroups that an XCD has of the cut tiles, 0 where it has the whole tile
    if (at < eights * row_wgs) {
        tile = at / row_wgs * 8 + xcd;
        wg = at - at / row_wgs * row_wgs;
    } else {
        const int32_t rest = (tiles - eights * 8) * row_wgs, i = xcd * ((rest + 7) / 8) + (at - eights * row_wgs);
        slice = (rest + 7) / 8;
        if (at - eights * row_wgs >= slice || i >= rest) return;     // the whole workgroup
        tile = eights * 8 + i / row_wgs;
        wg = i - i / row_wgs * row_wgs;
    }
    const RowsTile<LPR, WIDE, AHEAD, SUMS> T(a, tile);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t m = (int32_t)a.m, w0 = (wg * kRowsWaves + wv) * rpw;                    // the wave's first row
    const int32_t wrows = m - w0 < 0 ? 0 : (m - w0 < rpw ? m - w0 : rpw);
    const int32_t start = T.lane <= wrows && wrows > 0 ? a.row_ptr[w0 + T.lane] : 0;
    int32_t turn = wg;
    if constexpr (LONG == kLongSpread) turn = slice ? rows_turn(turns, wg) : wg;
    const int32_t long_first = PLACES && turn < a.long_room ? a.long_rows[turn] : -1;    // (asked for beside the starts)
    int32_t n_front = PLACES ? 0 : (a.long_count ? a.long_count[2] : 0), n_long = PLACES ? a.long_room : (a.long_count ? a.long_count[0] : 0);
    n_front = n_front < a.long_room ? n_front : a.long_room;
    n_long = n_long < a.long_room - n_front ? n_front + n_long : a.long_room;
    if (__builtin_expect(!PLACES && slice && n_long > 0, 0)) {
        // The XCDs that share a tile take its long rows in turns: by the place of a workgroup among those of its XCD, then by XCD.  (In the order of `wg` the first XCD of a tile would
        // have them all; power-law rows, 9958 x 11050, N = 64, 128, 256: 26.5 41.4 48.8 us so, 18.8 24.9 33.3 in turns.)
        const int32_t t0 = (tile - eights * 8) * row_wgs, t1 = t0 + row_wgs, from = xcd * slice > t0 ? xcd * slice : t0, before = t0 + wg - from;
        turn = 0;
        for (int32_t x = 0; x < 8; ++x) {
            const int32_t lo = x * slice > t0 ? x * slice : t0, hi = (x + 1) * slice < t1 ? (x + 1) * slice : t1, n = before + (x < xcd ? 1 : 0);
            if (hi > lo) turn += hi - lo < n ? hi - lo : n;
        }
    }
    // (out of the way of matrices without long rows; 12000 x 12000, 0.5 %, N = 64: level, 12.15 us without the hints, 12.13 so)
    if (PLACES || __builtin_expect(n_long > 0, 0)) rows_long_rows<LPR, WIDE, AHEAD, SUMS, LONG>(T, n_front, n_long, turn, row_wgs, long_first, part);
    rows_of_wave<LPR, WIDE, AHEAD, SUMS>(T, w0, wrows, start, wave_row, a.long_row);
}

// The whole product of a matrix with uneven rows by the first kRowsAllWgs workgroups of a launch whose workgroups have a compute unit each (gridDim.x is a multiple of 8).  An XCD walks one
// tile after the other, the tiles beyond the last whole eight are cut into a share of rows per workgroup.  A share is a stretch of rows with as many entries as the others (kRowsAllRow
// for a row itself), another one in every tile.  The waves of a workgroup take from one queue: first its long rows in kRowsPieces pieces each, then the other rows, `rpw` at a time.  The wave that
// ends the last piece of a row adds the sums of its pieces in their order, so that nobody waits for anybody and the bits are the same on every run.
// Power-law rows, us: 16384 x 16384, N = 1024: 430 as items of 64 rows, the long ones by all sixteen waves between two barriers, which nothing filled; 280 with the queue and equal numbers of rows;
// 257 with shares of equal entries; 189 with a workgroup on every compute unit whatever the bands ask for.  9958 x 11050, N = 1000: 506 -> 159; 17411 x 20000, N = 704: 415 -> 159.
constexpr int kRowsAllWgs = 256, kRowsPieces = 8, kRowsAllLong = 64, kRowsAllRow = 8;
struct RowsAllLds {
    float sums[kRowsAllLong * kRowsPieces][64];           // of the pieces of the long rows
    int32_t row[kRowsAllLong], beg[kRowsAllLong], end[kRowsAllLong], ended[kRowsAllLong], next, count;
};
// The first row r with row_ptr[r] + kRowsAllRow r of at least the part num / den of it all; by all lanes of a wave.
__device__ __forceinline__ int32_t rows_all_cut(const RowsArgs& a, int64_t num, int64_t den, int lane)
{
    const int64_t target = (a.nnz + kRowsAllRow * a.m) * num / den;
    int32_t lo = 0, hi = (int32_t)a.m;
    while (lo < hi) {
        const int32_t step = (hi - lo + 63) / 64;
        const int64_t at = (int64_t)lo + (int64_t)(lane + 1) * step - 1;
        const bool below = at < hi && (int64_t)a.row_ptr[at] + kRowsAllRow * at < target;
        const int32_t n = (int32_t)__popcll(__ballot(below));
        const int64_t top = (int64_t)lo + (int64_t)(n + 1) * step - 1;
        lo += n * step;
        hi = top < hi ? (int32_t)top : hi;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}
template <int LPR>
__device__ __forceinline__ void rows_all(const RowsArgs& a, int32_t tiles, int32_t rpw, int32_t wave_row, RowsAllLds& lds)
{
    static_assert(LPR * 4 <= 64, "the sums of a piece");
    const int32_t xcd = (int32_t)(blockIdx.x & 7u), place = (int32_t)(blockIdx.x >> 3), most = (int32_t)(gridDim.x >> 3), wgs = most < kRowsAllWgs / 8 ? most : kRowsAllWgs / 8;
    if (place >= wgs) return;                                          // the whole workgroup
    const int32_t eights = tiles / 8, rest = tiles - eights * 8, t = (int32_t)threadIdx.x, threads = (int32_t)blockDim.x;
    // the share [from, to) / parts of a tile
    auto tile_rows = [&](int32_t tile, int64_t from, int64_t to, int64_t parts) {
        const RowsTile<LPR, false, 16, 1> T(a, tile);
        const int32_t r0 = rows_all_cut(a, from, parts, T.lane), r1 = rows_all_cut(a, to, parts, T.lane);
        // its long rows: those of more entries than `limit`, which has room for all of them
        int32_t limit = kRowsPieces * 32, cnt;
        while (true) {
            __syncthreads();                                           // nobody is at the queue before, or at the count, any more
            if (t == 0) { lds.count = 0; lds.next = 0; }
            __syncthreads();
            for (int32_t r = r0 + t; r < r1; r += threads) {
                const int32_t lb = a.row_ptr[r], le = a.row_ptr[r + 1];
                if (le - lb > limit) {
                    const int32_t i = atomicAdd(&lds.count, 1);
                    if (i < kRowsAllLong) { lds.row[i] = r; lds.beg[i] = lb; lds.end[i] = le; lds.ended[i] = 0; }
                }
            }
            __syncthreads();
            cnt = __builtin_amdgcn_readfirstlane(lds.count);
            if (cnt <= kRowsAllLong) break;
            limit = limit < INT32_MAX / 2 ? 2 * limit : INT32_MAX;
        }
        const int32_t pieces = cnt * kRowsPieces, items = pieces + (r1 > r0 ? (r1 - r0 + rpw - 1) / rpw : 0);
        while (true) {
            int32_t q = 0;
            if (T.lane == 0) q = atomicAdd(&lds.next, 1);
            q = __builtin_amdgcn_readfirstlane(q);
            if (q >= items) break;
            if (q >= pieces) {
                const int32_t w0 = r0 + (q - pieces) * rpw, wrows = r1 - w0 < rpw ? r1 - w0 : rpw;
                // (a row above `limit` is taken out of the slots here, whatever `wave_row` is: it has its pieces)
                rows_of_wave<LPR, false, 16, 1>(T, w0, wrows, T.lane <= wrows ? a.row_ptr[w0 + T.lane] : 0, wave_row < limit ? wave_row : limit, limit);
                continue;
            }
            const int32_t i = q / kRowsPieces, piece = q % kRowsPieces;
            const int32_t r = __builtin_amdgcn_readfirstlane(lds.row[i]), lb = __builtin_amdgcn_readfirstlane(lds.beg[i]), le = __builtin_amdgcn_readfirstlane(lds.end[i]);
            constexpr int kSlots = 64 / LPR * kRowsPieces;
            const int32_t each = (le - lb + kSlots - 1) / kSlots, b = lb + (piece * (64 / LPR) + T.slot) * each, e = b + each < le ? b + each : le;
            const typename RowsTile<LPR, false, 16, 1>::Place pl = T.place(r);
            RowsAcc<1> sum = T.shared_row(pl, b, e);
            if (T.slot == 0)
#pragma unroll
                for (int u = 0; u < 4; ++u) lds.sums[q][T.sl * 4 + u] = sum.x[0][u];
            int32_t before = 0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (T.lane == 0) before = atomicAdd(&lds.ended[i], 1);
            before = __builtin_amdgcn_readfirstlane(before);
            if (before != kRowsPieces - 1) continue;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            if (T.slot == 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) sum.x[0][u] = lds.sums[i * kRowsPieces][T.sl * 4 + u];
                for (int s = 1; s < kRowsPieces; ++s)
#pragma unroll
                    for (int u = 0; u < 4; ++u) sum.x[0][u] += lds.sums[i * kRowsPieces + s][T.sl * 4 + u];
                T.store(r, pl, sum);
            }
        }
    };
    for (int32_t j = 0; j < eights; ++j) {
        const int32_t share = (place + j) % wgs;
        tile_rows(j * 8 + xcd, share, share + 1, wgs);
    }
    const int64_t all = 8 * wgs, from = ((int64_t)xcd * wgs + place) * rest, to = from + rest;        // of the other tiles, in parts of 1 / `all` of a tile
    for (int64_t x = from / all; x * all < to; ++x)
        tile_rows(eights * 8 + (int32_t)x, from > x * all ? from - x * all : 0, to < (x + 1) * all ? to - x * all : all, all);
}

template <int LPR, bool WIDE, int AHEAD, int SUMS, RowsLong LONG>
__global__ __launch_bounds__(kRowsThreads, AHEAD == 16 ? 4 : 8) void spdm_rows(RowsArgs a, int32_t tiles, int32_t row_wgs, int32_t rpw, int32_t wave_row, RowsTurns turns)
{
    __shared__ __attribute__((aligned(16))) float part[kRowsWaves][LPR * 4];
    rows_item<LPR, WIDE, AHEAD, SUMS, LONG>(a, blockIdx.x, tiles, row_wgs, rpw, wave_row, turns, part);
}

// B of one, two or three columns: sixteen lanes share a row, each takes every sixteenth entry, and their sums are added up in a
// fixed tree.
template <int N>
__global__ __launch_bounds__(kRowsThreads) void spdm_vectors(RowsArgs a)
{
    const int lane = threadIdx.x & 15;
    const int64_t r = (int64_t)blockIdx.x * (kRowsThreads / 16) + (threadIdx.x >> 4);
    const uint32_t kmax = (uint32_t)(a.k - 1);
    float sum[N];
#pragma unroll
    for (int n = 0; n < N; ++n) sum[n] = 0.0f;
    if (r < a.m) {
        const int32_t end = a.row_ptr[r + 1];
        for (int32_t e = a.row_ptr[r] + lane; e < end; e += 16) {
            uint32_t c = (uint32_t)a.cols[e];
            c = c < kmax ? c : kmax;
            const float v = a.vals[e];
            const float* b = a.B + (int64_t)c * a.ldb;
#pragma unroll
            for (int n = 0; n < N; ++n) sum[n] = __builtin_fmaf(v, b[n], sum[n]);
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) sum[n] += __shfl_xor(sum[n], d, 16);
    if (r < a.m && lane == 0)
#pragma unroll
        for (int n = 0; n < N; ++n) a.C[r * a.ldc + n] = sum[n];
}

}  // namespace gcoo
