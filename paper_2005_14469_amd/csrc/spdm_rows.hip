// The row-by-row SpDM kernel and its launcher.
#include "gcoo_spdm_rows_kernel.hpp"

namespace gcoo {

template <int LPR, bool WIDE = false>
static hipError_t launch_rows(const RowsArgs& a, hipStream_t s)
{
    constexpr int64_t waves = kRowsThreads / 64, tile = 4 * LPR, spw = 64 / LPR;
    // rows of C that do not start at a 128-byte line: the tiles are moved down by up to 31 columns
    const bool aligned = a.ldc % 32 == 0 && reinterpret_cast<uintptr_t>(a.C) % 128 == 0;
    const int64_t tiles = (a.N + (aligned ? 0 : 31) + tile - 1) / tile, mean = a.nnz / a.m;
    auto groups = [&](int64_t r) { return (a.m + waves * r - 1) / (waves * r); };
    // Rows per wave: one per slot, so that a launch has many short workgroups.  Short rows (one batch each) go several to a
    // slot, the loads of one behind those of the one before, while enough workgroups are left (64 columns per tile, rows of 6 entries,
    // 12000 x 12000: 445 us with 4 rows per wave, 408 with 8, 399 with 16; rows of 12: 553, 499, 501; 12001 x 12001: 512, 471, 472 and
    // 683, 653, 708; rows of 25 to 80 entries are fastest with 4).  A launch that cannot
    // fill the chip has fewer rows per wave, each on all slots of it.
    int64_t rpw = spw;
    if (mean <= 12) {
        while (2 * rpw <= kShortRowsPerWave && groups(2 * rpw) * tiles >= 4096) rpw *= 2;
    } else {
        while (rpw > 1 && groups(rpw) * tiles < 256) rpw /= 2;
    }
    const int64_t row_wgs = groups(rpw);
    const int64_t rest = tiles % 8 * row_wgs, grid = tiles / 8 * 8 * row_wgs + (rest + 7) / 8 * 8;
    if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    // Rows well above the mean hold their slot up while the others of the wave have ended: all slots of the wave take them.
    const int64_t wave_row = rpw < spw ? 8 : (2 * mean > 64 ? 2 * mean : 64);
    const bool places = !a.long_count && a.long_room > 0;
    (places ? spdm_rows<LPR, WIDE, true> : spdm_rows<LPR, WIDE, false>)<<<dim3((unsigned)grid), dim3(kRowsThreads), 0, s>>>(
        a, (int32_t)tiles, (int32_t)row_wgs, (int32_t)rpw, (int32_t)(wave_row > INT32_MAX ? INT32_MAX : wave_row));
    return hipGetLastError();
}

hipError_t launch_spdm_rows(const RowsArgs& a, hipStream_t s)
{
    if (a.m < 1 || a.k < 1 || a.N < 1 || a.ldb > 0x3fffffffLL) return hipErrorInvalidValue;
    if (a.N < 4) {
        constexpr int64_t rows = kRowsThreads / 16;
        const int64_t grid = (a.m + rows - 1) / rows;
        if (a.N == 1) spdm_vectors<1><<<dim3((unsigned)grid), dim3(kRowsThreads), 0, s>>>(a);
        else if (a.N == 2) spdm_vectors<2><<<dim3((unsigned)grid), dim3(kRowsThreads), 0, s>>>(a);
        else spdm_vectors<3><<<dim3((unsigned)grid), dim3(kRowsThreads), 0, s>>>(a);
        return hipGetLastError();
    }
    // a B of more than 4 GB is beyond the offsets of a buffer descriptor
    if ((uint64_t)a.k * (uint64_t)a.ldb * 4u > kRowsMaxBytes) return launch_rows<16, true>(a, s);
    // 64, 32 or 16 columns per tile: the fewest lanes without a column of their own
    if (a.N <= 16) return launch_rows<4>(a, s);
    if (a.N <= 32) return launch_rows<8>(a, s);
    // 128 columns per tile while the tile stays in an XCD's L2 (4 MB): rows of B that do not start at 128-byte lines cost a line
    // more per segment (3000 x 3000, 1 %: N = 2999 59.9 us with 64 columns, 50.9 with 128; 9001 columns: 452 and 460).
    // Rows of a few entries take theirs from a tile of B hardly more than once before it has to be read anyway, so that the wider
    // stretches of B and C count for more than the L2 while C is wide (us with 16, 32, 64 lanes; 12000 x 12000, rows of 1, 3, 5, 9 entries:
    // 339 277 249, 373 328 311, 398 364 374, 446 440 568; 14000 rows, N = 2000, of 3, 5, 7: 80 71 69, 86 79 85, 93 94 108; N = 501, of 3: 22 28 30;
    // 3000 x 3000, of 3: 22 21 25).
    // Where between two points of these sweeps a line lies is a choice, not derived from anything.
    const bool lines = a.ldb % 32 == 0 && reinterpret_cast<uintptr_t>(a.B) % 128 == 0;
    if (a.N >= 1500 && a.nnz <= 4 * a.m && a.m * a.N >= 20000000) return launch_rows<64>(a, s);
    if (a.N > 64 && (a.k <= (lines ? 4096 : 6500) || (a.N >= 1500 && a.nnz <= (a.N >= 6000 ? 9 : 6) * a.m))) return launch_rows<32>(a, s);
    return launch_rows<16>(a, s);
}

}  // namespace gcoo
