// Host-side launch interface of the SpDM kernels.  Each V (columns per lane) of the register kernel is compiled
// in a translation unit of its own (spdm_sched_v*.hip) so that the instances build in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

namespace gcoo {

struct SchedClass;

struct SpdmArgs {
    const SchedClass* hdr;     // [g][nw][kMaxRun]
    const uint32_t* stream;    // run schedule
    const int32_t* gIdxes;     // [g+1]
    int64_t m;
    int32_t p;
    int64_t g;
    int32_t nw;                // column windows of the schedule
    const float* B;
    int64_t ldb;
    int64_t N;
    float* C;
    int64_t ldc;
    int64_t nnz;
    // statistics of the conversion on the device ([1] = entries of the largest group), from which the
    // kernel derives the entry count from which a group is split over the waves of a workgroup; nullptr: the
    // launch has too many items for that to pay
    const unsigned long long* stats;
    // order[0..g): the groups by falling size; order[g..2g): those sizes.  nullptr: not built (more than
    // kOrderMaxGroups groups)
    const int32_t* order;
};

// V = 4 needs p <= 32, V = 38 (four columns per lane, tall accumulator file) p <= 38, V = 2 needs
// p <= 64; N at least the columns per lane, ldb < 2^30, any alignment of 4 bytes.
// Anything else returns hipErrorInvalidValue.
hipError_t launch_spdm_sched(int V, const SpdmArgs& a, hipStream_t s);

hipError_t launch_spdm_sched_v4(const SpdmArgs& a, hipStream_t s);
hipError_t launch_spdm_sched_v4_tall(const SpdmArgs& a, hipStream_t s);
hipError_t launch_spdm_sched_v2(const SpdmArgs& a, hipStream_t s);

// The workgroup-shared kernel that reads the share schedule: p <= 48; N, ldb, ldc multiples of 4; B and C
// 16-byte aligned; every row offset of B in bytes below 2^32.
struct ShareArgs {
    const uint32_t* hdr;       // headers
    const uint32_t* blocks;    // streams
    const int32_t* sbase;      // [8 * nq] first block of every stream
    const int32_t* ucols;      // distinct columns per super-group, the list of Q starting at gIdxes[8Q]
    const int32_t* ucount;     // [nq]
    const int32_t* gIdxes;     // [g + 1]
    int64_t m;
    int32_t p;
    int64_t g;
    int64_t nq;                // super-groups
    const float* B;
    int64_t ldb;
    int64_t N;
    float* C;
    int64_t ldc;
};
hipError_t launch_spdm_share(const ShareArgs& a, hipStream_t s);

// Which place workgroup `wg` of a tile begins with, where XCDs share the tile and the long rows are in places of a dense matrix: a stretch of a tile's workgroups is on one XCD, and the places in
// their order would be too.  The workgroups are cut into as many pieces as XCDs share a tile, and the places are dealt to the pieces one by one.  Product against a counted list, places in their order and so:
// twenty rows 90 % full in matrices of rows of a few entries, 31 of 1000 to 20000 rows, N = 16 to 1000: 1.05 0.98 of the time (us: 2564 x 1762, N = 120: 11.8 15.8 11.5); power-law rows, 59 of them: 1.00 1.01; even rows: 0.98 0.98.
// (Exact turns by XCD, a sum over the XCDs in front of the entries: even rows 1.02.  From CSR arrays, where long rows are in places too, 166 uneven matrices were level with and without.)
struct RowsTurns {
    int32_t piece, whole, rest;      // workgroups of a piece, pieces of as many, workgroups of the one behind them
    uint32_t inverse;                // of `piece`, in units of 2^-32
};
constexpr int64_t kRowsTurnsMost = 65535;      // workgroups of a tile up to which the quotient below is exact: its error is less than wg x piece in 2^-32 of one
inline RowsTurns rows_turns(int64_t row_wgs, int64_t tiles)
{
    const int64_t rest = tiles % 8 ? tiles % 8 : 8, xcds = (8 + rest - 1) / rest, even = (row_wgs + xcds - 1) / xcds, piece = even > 2 ? even : 2;
    return {(int32_t)piece, (int32_t)(row_wgs / piece), (int32_t)(row_wgs % piece), (uint32_t)(0xffffffffull / (uint64_t)piece) + 1u};
}
__host__ __device__ inline int32_t rows_turn(const RowsTurns& t, int32_t wg)
{
    const int32_t q = (int32_t)(((uint64_t)(uint32_t)wg * t.inverse) >> 32), i = wg - q * t.piece;
    return i < t.rest ? i * (t.whole + 1) + q : t.rest * (t.whole + 1) + (i - t.rest) * t.whole + q;
}

// The kernel that works row by row on the entries in row order: any N, ldb < 2^30, any alignment of 4 bytes, k >= 1.
struct RowsArgs {
    const int32_t* row_ptr;    // [m + 1]
    const int32_t* cols;       // [nnz]
    const float* vals;         // [nnz]
    int64_t m;
    int64_t k;
    int64_t nnz;
    const float* B;
    int64_t ldb;
    int64_t N;
    float* C;
    int64_t ldc;
    const int32_t* long_rows;  // long_room places for the rows of more than `long_row` entries (RowsOut)
    const int32_t* long_count; // or null: -1 in places without a row
    int32_t long_row, long_room;
    int32_t moved;             // 31: tiles are moved down to whole lines of C, 0: they are not (set by the launchers)
};
// A row of more entries than this is shared by a whole workgroup.
inline int32_t rows_long(int64_t m, int64_t nnz)
{
    const int64_t n = m > 0 ? 8 * (nnz / m) : 0;
    return (int32_t)(n < 512 ? 512 : (n > INT32_MAX ? INT32_MAX : n));
}
// By how many columns at the most the tiles are moved down, so that the rows of C are stored in whole 128-byte lines.  That costs a tile more and, where B has the pitch of C, takes nothing from
// the lines of B that a stretch lies in: it pays where C is most of the traffic (us, moved and not: 12471 x 12471, rows of 1.1 entries, N = 5125: 76 81; 10845 columns, rows of 5.3, N = 9494:
// 343 350; 6298, of 7.2, N = 2285: 42 38; 11050, of 44, N = 237: 45 37).  From 129 to 160 columns there are three tiles of 64 either way, and the last is not a sliver (over 65 products 2 to 3 % less:
// 18677 x 20000, of 13.5, N = 155: 23.5 25.7; power-law rows, 14575 x 13587, N = 158: 65 71; but from 65 to 97 level).
inline int32_t rows_moved(int64_t m, int64_t nnz, int64_t N, const float* C, int64_t ldc)
{
    if (ldc % 32 == 0 && reinterpret_cast<uintptr_t>(C) % 128 == 0) return 0;
    return nnz <= 4 * m || (nnz <= 8 * m && m * N >= 25000000) || (N > 128 && N <= 160) ? 31 : 0;
}
// Largest B (k x ldb) whose rows a buffer descriptor reaches with something left above for the entries past the end of a row.
constexpr uint64_t kRowsMaxBytes = 0xffffefffull;
// `spread`: long rows in places are taken by rows_turn().
hipError_t launch_spdm_rows(const RowsArgs& a, bool spread, hipStream_t s);

// The kernel that works row by row on a tile of B in LDS (gcoo_spdm_tile_kernel.hpp), `row_wgs` workgroups per tile of kTileCols columns: N of at least a tile, any alignment of
// 4 bytes, at most kTileMaxRows rows for a workgroup, tile_lds() at most kTileLdsBytes, k x ldb at most kRowsMaxBytes, at most kTileMaxNnz entries.
constexpr int kTileCols = 16;
constexpr int kTileMaxRows = 1023;
constexpr int64_t kTileLdsBytes = 160 * 1024 - 16;        // the kernel has two words of its own
constexpr int64_t kTileMaxNnz = 1 << 29;                  // byte offsets of entries
constexpr int kTileBins = 256;                            // lengths of rows in steps of four entries; the last bin is open
// Its LDS: the tile, k rows of B and one of zeros, and before it comes in, in the same place, the bins of the row lengths; behind the larger of the two (the bins up to 14 columns), where
// the workgroup's rows begin, `rows` + 1; its rows by falling length, 16 bits each.
constexpr int64_t tile_lds_rows(int64_t k) { return (k + 1) * (4 * kTileCols) > 4 * kTileBins ? (k + 1) * (4 * kTileCols) : 4 * kTileBins; }
constexpr int64_t tile_lds(int64_t k, int64_t rows) { return tile_lds_rows(k) + 4 * (rows + 1) + 2 * rows; }
constexpr int64_t tile_most_rows(int64_t k)               // of a workgroup; less than 1: the kernel does not serve so many columns
{
    const int64_t room = (kTileLdsBytes - 4 - tile_lds_rows(k)) / 6;
    return room < kTileMaxRows ? room : kTileMaxRows;
}
hipError_t launch_spdm_rows_tile(const RowsArgs& a, int64_t row_wgs, bool whole, hipStream_t s);


// The sixteen-wave kernel that reads the band schedule (gcoo_band.hpp): N of at least a tile, or N, ldb a multiple of 4 and B 16-byte aligned; a B of at
// most kRowsMaxBytes (the launch may work row by row).
struct BandArgs {
    const uint32_t* head;
    const uint32_t* units;
    const int32_t* first;      // [16 * blocks] first unit of every wave
    const int32_t* count;      // [blocks] distinct columns
    int32_t blocks;
    int32_t h;                 // rows per wave
    int32_t v;                 // columns per lane: 4 (the wide cut) or 2 (the tall one)
    int32_t total, grid;       // workgroups with work, workgroups launched (set by the launcher)
    const uint32_t* uneven;    // not 0: no schedule was built, the rows are multiplied one by one
    int64_t head_stride;
    int64_t m;
    int64_t k;
    const float* B;
    int64_t ldb;
    int64_t N;
    float* C;
    int64_t ldc;
};
// `rows` is for a matrix whose rows turn out to be uneven.
hipError_t launch_spdm_band(const BandArgs& a, const RowsArgs& rows, hipStream_t s);

}  // namespace gcoo
