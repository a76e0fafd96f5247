// The row-by-row SpDM kernel and its launcher.
#include "gcoo_spdm_rows_kernel.hpp"

namespace gcoo {

// Waves of a launch that has one row and 256 columns to each: 8192 are resident at a time.
static int64_t rows_waves(int64_t m, int64_t N) { return m * ((N + 255) / 256); }

template <int LPR, bool WIDE, int AHEAD, int SUMS>
static hipError_t launch_rows_ahead(const RowsArgs& args, bool spread_places, hipStream_t s)
{
    constexpr int64_t waves = kRowsThreads / 64, tile = 4 * LPR, spw = 64 / LPR;
    RowsArgs a = args;
    a.moved = rows_moved(a.m, a.nnz, a.N, a.C, a.ldc);
    const int64_t tiles = (a.N + a.moved + tile - 1) / tile, mean = a.nnz / a.m;
    auto groups = [&](int64_t r) { return (a.m + waves * r - 1) / (waves * r); };
    // Rows per wave: one per slot, so that a launch has many short workgroups, and two or four per slot where rows are short, the loads of one behind those of the one before
    // (us, 1, 2, 4, 8 and 16 rows per wave: 7999 x 7999, rows of 8, 64 columns per tile - 231 169 177 229, 128 columns - 164 176 211 261; 12001 x 12001, of 6, 128 columns
    // - 426 426 448 482; 5000 x 5000, of 2, N = 5001, 256 columns - 42.6 43.2 46.1 46.3).  Not where all waves are resident at once: there a row more is a trip to memory more (322 x 295, of 2,
    // N = 295, kernel alone, 2 and 4 rows: 3.2 3.9).  A launch of fewer than 192
    // workgroups has a row per wave, on all slots of it.  (Rows of more than 12 entries, a row and four rows per wave: 0.83 to 0.98 of the time below 125 workgroups, 0.94 to 1.02 up to 200, 1 to 1.05 up to
    // 256; two rows per wave, each on half of the slots, never less than the better of the two.  By eight lanes, 8123 x 11104, rows of 13, N = 22: eight rows per wave 5.3 us, four 7.3.)
    int64_t rpw = spw;
    const bool many = rows_waves(a.m, a.N) > 8192;
    if (many && mean < 6) rpw = LPR == 32 ? 4 : (LPR == 64 ? 2 : spw);
    else if (many && mean < 10) rpw = LPR == 64 ? 2 : spw;
    else if (mean >= 120 && groups(rpw) * tiles < 4096) rpw = spw > 4 ? spw / 4 : 1;         // (9072 x 9072, rows of 143, N = 34: 19.0 16.3; 17015, of 279, N = 20: 51.5 40.6)
    else if (mean > 12 && groups(rpw) * tiles < 192) rpw = 1;
    const int64_t row_wgs = groups(rpw);
    const int64_t rest = tiles % 8 * row_wgs, grid = tiles / 8 * 8 * row_wgs + (rest + 7) / 8 * 8;
    if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    // Rows well above the mean hold their slot up while the others of the wave have ended: all slots of the wave take them.
    const int64_t wave_row = rpw < spw ? 8 : (2 * mean > 64 ? 2 * mean : 64);
    const bool places = !a.long_count && a.long_room > 0;
    const bool spread = places && spread_places && tiles % 8 && row_wgs <= kRowsTurnsMost;
    const auto kernel = !places ? spdm_rows<LPR, WIDE, AHEAD, SUMS, kLongCounted> : (spread ? spdm_rows<LPR, WIDE, AHEAD, SUMS, kLongSpread> : spdm_rows<LPR, WIDE, AHEAD, SUMS, kLongPlaces>);
    kernel<<<dim3((unsigned)grid), dim3(kRowsThreads), 0, s>>>(a, (int32_t)tiles, (int32_t)row_wgs, (int32_t)rpw, (int32_t)(wave_row > INT32_MAX ? INT32_MAX : wave_row),
                                                               spread ? rows_turns(row_wgs, tiles) : RowsTurns{});
    return hipGetLastError();
}

// A wave with eight rows of B in flight in place of sixteen needs half of the registers, so that twice as many waves are resident: faster where a row has not many more entries
// than that (us, sixteen and eight: 12001 x 12001, rows of 6: 437 426; 7999 x 7999, of 8: 187 164; 10643 x 10643, of 1.2, N = 8867: 157 125; over 318 products 12 to 20 % less below 6 entries
// per row, 2 to 9 % from 6 to 16, level from 16 to 30, 2 to 5 % more above, 13 % more for power-law rows of 49).
// SUMS: of a row in a slot (rows_fma()): as many as there are slots of 16 lanes in one, and two where 16 lanes serve up to 32 columns, for which eight are enough.
template <int LPR, int SUMS = LPR <= 16 ? 1 : LPR / 16>
static hipError_t launch_rows(const RowsArgs& a, bool spread, hipStream_t s)
{
    if constexpr (LPR >= 16)
        if (a.nnz <= 16 * a.m) return launch_rows_ahead<LPR, false, 8, SUMS>(a, spread, s);
    return launch_rows_ahead<LPR, false, 16, SUMS>(a, spread, s);
}

hipError_t launch_spdm_rows(const RowsArgs& a, bool spread, hipStream_t s)
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
    if ((uint64_t)a.k * (uint64_t)a.ldb * 4u > kRowsMaxBytes) return launch_rows_ahead<16, true, 16, 1>(a, spread, s);
    // Up to 32 columns: four or eight lanes to a row where that leaves enough workgroups, sixteen else, those without a column of their own along (kernel alone, us, 8 lanes and 16:
    // 6124 x 6124, rows of 19, N = 28: 7.4 4.9; 8788 x 9414, of 18, N = 27: 5.6 6.2).
    if (a.N <= 32 && a.m >= 7000) return a.N <= 16 && a.m >= 16384 ? launch_rows<4>(a, spread, s) : launch_rows<8>(a, spread, s);
    if (a.N <= 32) return launch_rows<16, 2>(a, spread, s);
    // ("As many entries as uneven rows have on average" below: the host knows the mean only, and 25 to 90 entries is that of the power law that was measured, exponent 1.5 with up to 4096 entries, over 2000 to 20000 columns.
    // Uniform rows of such a mean lose by it, up to 30 % between 129 and 400 columns; power-law rows of another exponent or limit have another mean.)
    // 64, 128 or 256 columns per tile.  Wider tiles are fewer requests for the same bytes and, where rows of B begin inside a 128-byte line, fewer lines per byte (3 for
    // 256 bytes, 5 for 512, 9 for 1024); narrower ones stay in an XCD's L2 (4 MB) at more rows of B, and have more slots to a wave for uneven rows, of which the host knows nothing.
    // From the times of all three in 960 products with rows of B inside a line and 800 with rows on lines, 300 to 20000 rows and columns, rows of 1 to 250 entries and power-law rows (us,
    // 64, 128, 256 columns): N below 1000: power-law rows, 4281 x 5127, N = 512: 26 35 57; even rows of 25 to 90 entries lose 2 to 9 % by 64 columns; 11050 x 11050, rows of 44, N = 86: 20 14.  Rows of a few entries
    // hardly take a row of B more than once before it has to be read anyway: 10643 x 10643, of 1.2, N = 8867: 201 170 157; 18739 rows of 5.6, N = 5569: 355 340 354; 12862 of 9.3, N = 2461: 133 144
    // 160.  Few columns: 3494 x 3494, rows of 12.6, N = 5853: 91 81 75; 4366 columns, N = 10409: 237 211 220.  Where between two points of these sweeps a line lies is a choice.
    const bool lines = a.ldb % 32 == 0 && reinterpret_cast<uintptr_t>(a.B) % 128 == 0;
    // While all waves are resident at once, 256 columns to each are the shortest way (kernel alone, us, 64, 128 and 256 columns: 408 x 408, rows of 0.3, N = 583: 3.4 3.4 3.3; 639 x 796, of 21,
    // N = 639: 6.0 5.7 5.0; 2217 x 1707, of 22, N = 197: 7.3 6.4 5.4; over 96 products 5 to 10 % less), but for up to 128 columns and for rows of as many entries as uneven ones have on average.
    const int64_t waves = rows_waves(a.m, a.N);
    // From half of those waves on only where the last tile is not mostly empty (three matrices in turn, 64, 128 and 256 columns: 2350 x 2350, of 5, N = 317: 4.7 5.0 5.9; 2176 x 2068, of 5, N = 456: 4.9 5.0 5.5;
    // 4006 x 5846, of 12, N = 302, as the rules below have it and 256: 9.0 11.9; but 1541 x 1249, of 3, N = 466: 4.0 4.1 4.0; one tile, 4106 x 2467, of 25, N = 204: 10.2 8.5).
    const bool full = waves <= 4096 || a.N <= 256 || 256 * 100 * ((a.N + 255) / 256) <= 115 * a.N;
    // Nor for rows of 28 entries and more on less than 600 waves, 700 from 36 on: 64 columns and all slots of a wave on a row take 0.89 to 0.97 of the time for rows of 36 and more, 0.97 for 28 to 36, but 1.00 to 1.07 at 700 to
    // 1000 waves, and 1.02 and 1.06 for rows of 20 to 28 and of 14 to 20 (300 products, three matrices in turn; us: 221 x 221, rows of 41, N = 235: 4.7 and 4.15; 250 x 377, of 58, N = 250: 5.3 and 4.7).
    const bool sparse_launch = a.nnz >= 28 * a.m && waves < (a.nnz >= 36 * a.m ? 700 : 600);
    // Nor for rows of 36 entries and more on 1025 to 1399 waves, that is 257 to 350 workgroups, whose last tile is more than a quarter empty: a compute unit with a second workgroup has eight long chains, and a part of them works for
    // nothing, where tiles of 64 columns are workgroups enough to come out even (39 products, three matrices in turn, 13 % less by 64 columns, up to 1199 waves 16 %, above 8 %; us, 256 and 64: 530 x 530, rows of 95, N = 267: 8.9 6.6;
    // 363 x 363, of 68, N = 547: 7.55 6.1; 590 x 590, of 39, N = 335: 5.8 5.4; with less of the tile empty 0.87 to 1.11 in 11 others, from 1400 waves on 0.92 to 1.02).
    const bool uneven_rounds = a.nnz >= 36 * a.m && waves > 1024 && waves < 1400 && a.N < 192 * ((a.N + 255) / 256);
    // Nor for many rows of B on lines, where wider tiles take no fewer lines per byte and B leaves an XCD's L2 the sooner (time against 64 columns, rows of 3 to 25 entries, 700 products: up to 1000 rows of B 0.90 to 0.97, to 1500
    // 0.93 to 1.05, to 2500 0.97 to 1.02 for N up to 256 and 1.01 to 1.20 beyond, from there on 1.01 to 1.25: 5000 to 8192 rows of B, rows of 10 to 25, N = 224 and 256: 1.22).
    const bool stays = !lines || a.k <= (a.N <= 256 ? 2500 : 1500);
    if (a.N > 64 && waves <= 8192 && full && !sparse_launch && !uneven_rounds && stays && (a.nnz < 25 * a.m || a.m < 1000))
        return a.N > 128 || (waves < 1000 && a.nnz < 25 * a.m) ? launch_rows<64>(a, spread, s) : launch_rows<32>(a, spread, s);
    if (a.N >= 1500 && a.nnz <= 3 * a.m && a.m * a.N >= 20000000) return launch_rows<64>(a, spread, s);
    // From 897 columns on there are eight tiles of 128 columns, one per XCD (us, 64 and 128 columns: power-law rows, 3611 x 3611, N = 926: 54 43; 4658 x 4658, N = 994: 64 56; 9046 x 9046, N = 895: 136 138;
    // rows of 89, 3454 x 3454, N = 917: 68 59; but power-law rows, 4830 x 7014, N = 663: 59 71; 8809 x 8809, N = 761: 103 126).
    if (a.N <= 896) {
        // One tile in place of three or four where rows begin inside lines: for rows of more entries than uneven ones have on average, while the tile stays near an XCD's L2, and up to 160 columns also where none of
        // the tiles would stay in it (us, 64 and 256 columns: 5699 x 6659, rows of 104, N = 134: 31 23; 8516 x 6585, of 65, N = 157: 28 22; 14161 x 14161, of 74, N = 154: 63 60; 5619 x 6520, of 55, N = 200: 20 17;
        // 12411 x 12959, of 20, N = 131: 17.3 15.2; 19195 x 15201, of 4, N = 148: 9.1 8.3; power-law rows, of 50, 17075 x 17075, N = 150: 89 78, 18289 x 20000, N = 130: 101 79; but 17686 x 17757, N = 151: 90 100, 9627 x 11477, of 84, N = 179: 46 50;
        // power-law rows, 2808 x 3141, N = 131: 17 37; 15071 x 15071, N = 131: 71 78).
        if (!lines && a.N > 128 && !sparse_launch) {
            const int64_t from = a.nnz >= 53 * a.m ? 0 : (a.nnz < 25 * a.m ? 11000 : (a.N <= 150 ? 16000 : INT64_MAX));
            if (a.N <= 160 ? a.k >= from : (a.N <= 208 && from == 0 && a.k <= 9100)) return launch_rows<64>(a, spread, s);
        }
        // one tile in place of two, and up to eight in place of sixteen, but not for rows of as many entries as uneven ones have on average (25 to 64 and 25 to 90; us, 64 and 128 columns:
        // 6133 x 5725, rows of 108, N = 93: 19.7 14.4; 6470 x 6470, of 98, N = 67: 20.8 15.5; over 40 products of rows of 64 and more, N = 65 to 128, up to 6500 rows of B, 13 % less)
        const bool one = !lines && a.N > 64 && a.N <= 128 && (a.k >= 6500 || a.nnz < 25 * a.m || a.nnz >= 64 * a.m), eight = a.N >= 700 && a.k <= 6500 && (a.nnz < 25 * a.m || a.nnz >= 90 * a.m);
        // and, for rows of 64 entries and more, wherever tiles of 128 columns are no wider together than those of 64 (up to 6500 rows of B: 0.83 to 0.95 of the time in 28 products of N = 209 to 512; where the last tile
        // would be half empty 0.98 to 1.3 in 40 others; us, 64 and 128 columns: 3218 x 3218, rows of 93, N = 326: 28.4 24.0)
        const bool even = !lines && a.nnz >= 64 * a.m && a.m >= 1000 && a.k < 6500 && (a.N - 1) % 128 >= 64;
        return one || eight || even || (a.N >= 200 && a.nnz <= 3 * a.m) ? launch_rows<32>(a, spread, s) : launch_rows<16>(a, spread, s);
    }
    if (a.N >= 1100 && a.k <= (lines ? 2600 : 3200)) return launch_rows<64>(a, spread, s);
    // Many rows of B: while all of B stays in the memory-side cache (256 MB), tiles of 64 columns, which stay longest in an XCD's L2; beyond, rows of a few entries take theirs from memory either way, and
    // in longer stretches by 128 columns (64 and 128; B inside lines: 12878 x 12878, rows of 6.1, N = 1563: 57 69; 13474 x 13474, of 4.5, N = 3602: 115 127; 10081 x 10081, of 4.4, N = 5285: 109 119; 8667 x 8667, of 6.5,
    // N = 6681: 138 144; but of 1.7 entries, 7706 x 8902, N = 1171: 19.3 16.6; of 4, 9739 x 9739, N = 1024: 19.4 17.8; 14065 x 14065, of 4, N = 6254: 236 212; 9307 x 9307, of 8.2, N = 9307: 320 283; 9531 x 9531, of 9.4: 357 322.  On lines: 13211 x 13211, of 3.8, N = 3584: 74 83; 10176 x 10176, of 4.6,
    // N = 10176: 250 233; 10372 x 12632, of 5.8, N = 10368: 288 273; 14533 x 14533, of 8.2, N = 14528: 576 626).
    const bool cached = a.k * a.N <= 66000000;
    const int64_t few = cached ? (a.N <= 1024 ? (lines ? 4 : 7) : 3) : (lines ? 6 : 10);          // entries per row; up to 1024 columns are eight tiles of 128
    if (a.k <= (cached ? 8000 : 9000) || a.nnz <= few * a.m) return launch_rows<32>(a, spread, s);
    return launch_rows<16>(a, spread, s);
}

}  // namespace gcoo
