// SpDM kernel that works row by row on a tile of B in LDS: C(r, :) = sum over the stored entries of row r of value x B(column, :), for matrices of so few
// columns that sixteen columns of the whole of B fit the LDS of a compute unit (k <= 2500 or so).
//
// The kernel that works row by row from the caches (gcoo_spdm_rows_kernel.hpp) has every entry's stretch of B come through the vector cache of its
// compute unit, 64 bytes per clock.  Here a workgroup of sixteen waves brings its columns of B into LDS once, for up to kTileMaxRows rows of A, and its entries take
// theirs from there: LDS gives four times as much per clock.
//
//   slot      four lanes x four adjacent columns, one row of A at a time: sixteen rows to a wave
//   entries   sixteen of a row at a time, four (column, value) pairs per lane; a DPP broadcast inside the quad hands each to the four lanes.
//             Per entry of sixteen rows: an address add, a read of LDS, a move and four multiply-adds, all from vector registers (a multiply-add with a DPP operand
//             would take twice as long)
//   order     the slots of a wave go through their rows side by side, so the workgroup puts its rows in the order of their lengths first, while the tile of B is
//             on its way; waves take the next sixteen as they come free.  Which wave multiplies a row and beside which others changes nothing in its sum
//   long rows rows well above the mean come first and have a whole wave each: equal stretches for the slots, sums added in a fixed tree
//   ends      what lies past the end of a row has the value 0 and a row of zeros behind the tile as its row of B, so that a non-finite row of B that no entry
//             touches stays out of C
//
// Bound: sixteen lanes read LDS in a clock, that is four rows of 64 bytes wherever they lie, and four random rows need 2.1 turns of the 64 banks: 8.4 clocks per
// instruction where it takes four without conflicts.  2000 x 2000, 10 %: 50 us of that in 60.  Tiles of 32 columns (1.5 turns, half as many columns of A) were as
// fast (1000 x 1000, 20 %: 18.1 and 19.2 us), of 64 slower; rows in the order of the matrix, not of their lengths, 64 us for the former.
// Bringing the tile in is the other part: 3.3 us for 147 KB at 1777 x 2301.
// Product alone, from the caches -> so (us): 1777 x 2301, 3 %, N = 1117: 27.6 -> 19.4; 2000 x 2000, 10 %: 122 -> 60; 2 %: 28 -> 19; 1000 x 1000, 5 %: 13.0 -> 9.3;
// 20 %: 40 -> 19.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcoo_spdm_launch.hpp"

namespace gcoo {

constexpr int kTileWaves = 16;
constexpr int kTileThreads = 64 * kTileWaves;
constexpr int kTileLanes = 4;                             // of a slot
constexpr int kTileSlots = 64 / kTileLanes;
constexpr int kTileRowBytes = 4 * kTileCols;              // of B, in LDS
constexpr int kTileLoads = 10;                            // 16-byte pieces of B per thread, at most
static_assert(kTileCols == 4 * kTileLanes && kTileMaxRows < kTileThreads && kTileLoads * kTileThreads * 16 >= kTileLdsBytes, "a thread per row and its end; all of the LDS");
typedef float tile_f32x4 __attribute__((ext_vector_type(4)));
typedef float tile_f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t tile_u32x4 __attribute__((ext_vector_type(4)));

// Pair i of a batch of 16 in every lane of the quad, whose lane i / 4 holds it in register i % 4.
template <int I>
__device__ __forceinline__ uint32_t tile_bcast(const uint32_t (&x)[4])
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[I % 4], (I / 4) * 0x55, 0xf, 0xf, true);       // quad_perm:[i/4,i/4,i/4,i/4]
}

struct TileBatch {
    uint32_t c[4], v[4];
    // 16 entries from `base` on; a load beyond the arrays returns zero, and what lies past the row's end is replaced by offsets()
    __device__ __forceinline__ void request(__amdgpu_buffer_rsrc_t cols, __amdgpu_buffer_rsrc_t vals, int32_t base, int lane)
    {
        const int at = (int)((uint32_t)(base + (lane & 3) * 4) * 4u);
        const tile_u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(cols, at, 0, 0), y = __builtin_amdgcn_raw_buffer_load_b128(vals, at, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) { c[j] = x[j]; v[j] = y[j]; }
    }
    // columns (beyond the last row of B they are brought inside: a device CSR input is not checked) -> places in LDS
    __device__ __forceinline__ void offsets(int32_t left, uint32_t kmax, int lane)
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = (lane & 3) * 4 + j < left;
            const uint32_t col = c[j] < kmax ? c[j] : kmax;
            c[j] = (in ? col : kmax + 1u) * (uint32_t)kTileRowBytes;
            v[j] = in ? v[j] : 0u;
        }
    }
};

// Entries I .. I + 3 of the batch.  (Eight reads of LDS in front of the multiply-adds need more than 64 registers: 1 to 5 % slower.)
template <int I>
__device__ __forceinline__ void tile_step(const TileBatch& b, const char* at, float (&acc)[4])
{
    tile_f32x4 x[4];
#define TILE_READ(J) x[J] = *reinterpret_cast<const tile_f32x4*>(at + tile_bcast<I + J>(b.c));
    TILE_READ(0) TILE_READ(1) TILE_READ(2) TILE_READ(3)
#undef TILE_READ
#define TILE_FMA(J)                                                                                          \
    {                                                                                                        \
        uint32_t w = tile_bcast<I + J>(b.v);                                                                 \
        asm("" : "+v"(w));                     /* a move of its own, not four multiply-adds with DPP */      \
        for (int u = 0; u < 4; ++u) acc[u] = __builtin_fmaf(__uint_as_float(w), x[J][u], acc[u]);            \
    }
    TILE_FMA(0) TILE_FMA(1) TILE_FMA(2) TILE_FMA(3)
#undef TILE_FMA
}

// Adds the entries [beg, end) of the slot's row.  `next` holds the first batch already; on return it holds the one at `more`, requested in front of the last entries.
__device__ __forceinline__ void tile_entries(__amdgpu_buffer_rsrc_t cols, __amdgpu_buffer_rsrc_t vals, TileBatch& next, int32_t beg, int32_t end, int32_t more, uint32_t kmax,
                                             const char* at, int lane, float (&acc)[4])
{
    int32_t left = end - beg;
    while (true) {
        TileBatch now = next;
        beg += 16;
        const bool last = !__any(left > 16);
        next.request(cols, vals, last ? more : beg, lane);
        now.offsets(left, kmax, lane);
        tile_step<0>(now, at, acc);
        if (__any(left > 4)) {
            tile_step<4>(now, at, acc);
            if (__any(left > 8)) {
                tile_step<8>(now, at, acc);
                if (__any(left > 12)) tile_step<12>(now, at, acc);
            }
        }
        if (last) return;
        left -= 16;
    }
}

// LDS: tile_lds_rows(), the bins where the tile comes to be.  Workgroup: (tile, rows [wg * rows, ...)), an XCD takes a stretch of them with the tiles side by side, so that the workgroups that read a
// line of B do so through one L2.  `long_steps`: a row of more steps of four entries than this has a wave to itself.
__global__ __launch_bounds__(kTileThreads, 8) void spdm_rows_tile(RowsArgs a, int32_t row_wgs, int32_t rows, int32_t total, int32_t long_steps)
{
    extern __shared__ __attribute__((aligned(16))) char tile_smem[];
    __shared__ int32_t counts[2];                                  // long rows, items taken
    const int32_t per = (int32_t)(gridDim.x >> 3), block = (int32_t)(blockIdx.x & 7u) * per + (int32_t)(blockIdx.x >> 3);
    if (block >= total) return;                                    // the whole workgroup
    const int32_t tile = block / row_wgs, wg = block - tile * row_wgs, n = (int32_t)a.N;
    // the last tile of a B that is no multiple of a tile wide begins where it can hold a whole one
    const int32_t j0 = tile * kTileCols, jb = j0 > n - kTileCols ? n - kTileCols : j0;
    const int32_t t = (int32_t)threadIdx.x, lane = t & 63, k = (int32_t)a.k, pieces = k * kTileLanes;
    const int64_t r0 = (int64_t)wg * rows;
    const int32_t mine = (int32_t)(a.m - r0 < rows ? a.m - r0 : rows);
    int32_t* row_at = reinterpret_cast<int32_t*>(tile_smem + tile_lds_rows(k));
    uint16_t* order = reinterpret_cast<uint16_t*>(row_at + rows + 1);
    int32_t* bins = reinterpret_cast<int32_t*>(tile_smem);

    int32_t start = t <= mine ? a.row_ptr[r0 + t] : 0;
    // this workgroup's columns of B, on their way while its rows are put in order
    __amdgpu_buffer_rsrc_t B = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.B + jb), 0, (int)(uint32_t)((uint64_t)(a.k - 1) * (uint64_t)a.ldb * 4u + kTileRowBytes), 0x00027000);
    const uint32_t ldb4 = (uint32_t)a.ldb * 4u;
    tile_u32x4 piece[kTileLoads];
#pragma unroll
    for (int j = 0; j < kTileLoads; ++j) {
        const int32_t i = j * kTileThreads + t;
        if (j * kTileThreads < pieces)
            piece[j] = i < pieces ? __builtin_amdgcn_raw_buffer_load_b128(B, (int)((uint32_t)(i / kTileLanes) * ldb4 + (uint32_t)(i % kTileLanes) * 16u), 0, 0) : 0u;
    }
    {
        const int32_t most = (int32_t)a.nnz;
        start = start < 0 ? 0 : (start > most ? most : start);
        if (t <= mine) row_at[t] = start;
        if (t < kTileBins) bins[t] = 0;
        if (t < 2) counts[t] = 0;
        int32_t bin = 0, place = 0;
        __syncthreads();
        if (t < mine) {
            const int32_t len = row_at[t + 1] - start, steps = len > 4 * (kTileBins - 1) ? kTileBins - 1 : (len > 0 ? (len + 3) / 4 : 0);
            bin = kTileBins - 1 - steps;
            place = atomicAdd(&bins[bin], 1);
            if (steps > long_steps) atomicAdd(&counts[0], 1);
        }
        __syncthreads();
        if (t < 64) {
            int32_t c[kTileBins / 64], sum = 0;
#pragma unroll
            for (int i = 0; i < kTileBins / 64; ++i) { c[i] = bins[t * (kTileBins / 64) + i]; sum += c[i]; }
            int32_t before = sum;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) { const int32_t o = __shfl_up(before, d, 64); before += lane >= d ? o : 0; }
            before -= sum;
#pragma unroll
            for (int i = 0; i < kTileBins / 64; ++i) { bins[t * (kTileBins / 64) + i] = before; before += c[i]; }
        }
        __syncthreads();
        if (t < mine) order[bins[bin] + place] = (uint16_t)t;
        __syncthreads();
    }

    const int slot = lane / kTileLanes, sl = lane % kTileLanes;
    const char* at = tile_smem + sl * 16;
    const uint32_t kmax = (uint32_t)(k - 1);
    __amdgpu_buffer_rsrc_t cols = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.cols), 0, (int)(uint32_t)(a.nnz * 4), 0x00027000);
    __amdgpu_buffer_rsrc_t vals = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.vals), 0, (int)(uint32_t)(a.nnz * 4), 0x00027000);
    const int32_t jc = jb + sl * 4;                                // the lane's first column; it stores those from j0 on
    const int32_t n_long = counts[0], items = n_long + (mine - n_long + kTileSlots - 1) / kTileSlots;
    // What the slot does of item x of the workgroup: a long row, shared by the slots, or sixteen rows.  row < 0: nothing.
    struct Item { int32_t row, beg, end; };
    auto item_of = [&](int32_t x) {
        Item q = {-1, 0, 0};
        const int32_t i = x < n_long ? x : n_long + (x - n_long) * kTileSlots + slot;
        if (x >= items || i >= mine) return q;
        q.row = order[i];
        q.beg = row_at[q.row];
        q.end = row_at[q.row + 1];
        if (x < n_long) {
            const int32_t each = (q.end - q.beg + kTileSlots - 1) / kTileSlots, e = q.beg + (slot + 1) * each;
            q.beg += slot * each;
            q.end = e < q.end ? e : q.end;
        }
        return q;
    };
    int32_t x = __builtin_amdgcn_readfirstlane(t >> 6);
    Item now = item_of(x);
    TileBatch next;
    next.request(cols, vals, now.beg, lane);
    // (the bins have been read: behind the barrier above)
#pragma unroll
    for (int j = 0; j < kTileLoads; ++j) {
        const int32_t i = j * kTileThreads + t;
        if (i < pieces) *reinterpret_cast<tile_u32x4*>(tile_smem + (size_t)i * 16) = piece[j];
    }
    if (t < kTileLanes) *reinterpret_cast<tile_u32x4*>(tile_smem + (size_t)(pieces + t) * 16) = tile_u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    while (x < items) {
        int32_t x2 = 0;
        if (lane == 0) x2 = kTileWaves + atomicAdd(&counts[1], 1);
        x2 = __builtin_amdgcn_readfirstlane(x2);
        const Item then = item_of(x2);
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        tile_entries(cols, vals, next, now.beg, now.end, then.beg, kmax, at, lane, acc);
        if (x < n_long) {
#pragma unroll
            for (int d = kTileLanes; d < 64; d <<= 1)
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[u] += __shfl_xor(acc[u], d, 64);
        }
        if (now.row >= 0 && (x >= n_long || slot == 0)) {
            float* dst = a.C + (r0 + now.row) * a.ldc + jc;
            if (jc >= j0) {
                *reinterpret_cast<tile_f32x4_any*>(dst) = tile_f32x4{acc[0], acc[1], acc[2], acc[3]};
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (jc + u >= j0) dst[u] = acc[u];
            }
        }
        x = x2;
        now = then;
    }
}

}  // namespace gcoo
