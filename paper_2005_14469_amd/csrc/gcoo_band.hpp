// The band schedule: the kernel-private listing that the sixteen-wave SpDM kernel reads (gcoo_spdm_band_kernel.hpp).
//
// A block is kBandWaves x h consecutive rows of A, wave w of the workgroup owning rows [w*h, (w+1)*h) of it (the
// blocks have nothing to do with the groups of the format).  The distinct columns of a block, ascending, are cut into bands:
// the rows of B that are in LDS together, band b in buffer b mod 2.  Two cuts of the same registers and the same LDS (BandCut):
//     wide   h <= 24, tiles of 256 columns, bands of 80 rows of B
//     tall   h <= 48 and even, tiles of 128 columns, bands of 160 rows of B; k <= kBandTallMaxK
//
// Units.  The entries of one (wave, band) are listed in steps of four records, four steps to a unit of 128 bytes, which
// the kernel fetches into scalar registers.  A record is 8 bytes:
//     { value (fp32 bits), row inside the wave's rows | place of its B row in LDS << kPlaceShift }     place = (b mod 2) * kRows + slot
// The steps of a (wave, band) begin on a unit of their own.  First the pair steps: two pairs of entries of one column each
// (the second entry of a pair reuses the B values of the first, the reuse of Algorithm 2), then the single steps.
// Records without an entry hold value 0 and row kSink: they add zero into a partial sum that is never stored.  Every (wave,
// band) has at least one unit, so that the units of a wave follow each other without gaps.
//
// Order.  Columns ascend inside the pairs and inside the singles, rows ascend inside a column; the last row of a column
// with an odd count is the single.  A wave whose rows repeat a coordinate has singles only, in row order (from the first stretch of kBandChunk distinct columns
// on that holds a repeated one).
//
// Heads.  head[(block * 16 + w) * stride + i], i = 0 .. bands + 1, stride = band_head_stride(k, kRows): eight words
//     { the columns whose B rows wave w fetches for band i, in five words; pair steps, single steps of band i - 1; unused }
// wide: a column per word; tall: two, c | (the next one - c) << 16 (bands beyond the last repeat the last column).
// count[block] = distinct columns; first[block * 16 + w] = first unit of a wave: what the waves before it can need at the most.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace gcoo {

constexpr int kBandWaves = 16;
constexpr int kBandHeadWords = 8;
constexpr int kBandFetches = 5;          // requests of a wave for the rows of a band, 1 KB each
constexpr int kBandUnitWords = 32;       // 16 records
constexpr int kBandSlackUnits = 2;       // read-ahead behind the last unit
constexpr int64_t kBandMaxK = 262144;    // the column bitmaps of a block are held in LDS
constexpr int64_t kBandTallMaxK = 65536; // a column and the distance to the next one share a word of the head

// V columns per lane: 4 is the wide cut, 2 the tall one.  (kMaxH + 1) x V partial sums per lane in v[28:127].
template <int V>
struct BandCut {
    static constexpr int kMaxH = 96 / V;
    static constexpr int kSink = kMaxH;
    static constexpr int kTile = 64 * V;
    static constexpr int kRows = 320 / V;
    static constexpr int kPlaceShift = V == 4 ? 10 : 9;          // a row of B in LDS is 256 V bytes
};
__host__ __device__ inline int band_rows_of(int v) { return 320 / v; }

// A list of more entries than this makes the matrix an uneven one, for which no schedule is built: the sixteen waves wait for each other
// in every band, so a list of three times the mean has the others wait two thirds of the time.  Uniform lists stay far below (960
// entries +- 31 at 8000 x 8000, 0.5 %).
inline int32_t band_heavy(int64_t nnz, int64_t lists)
{
    const int64_t n = lists > 0 ? 3 * (nnz / lists) + 512 : 0;
    return (int32_t)(n > INT32_MAX ? INT32_MAX : n);
}
// The column bitmaps that the schedule is built from: lists of up to 24 rows, one or two per wave.
__host__ __device__ inline int band_lists_of(int v) { return 4 / v; }
__host__ __device__ inline int64_t band_blocks(int64_t m, int32_t h) { return (m + kBandWaves * h - 1) / (kBandWaves * h); }
inline int64_t band_lists(int64_t m, int32_t h, int v) { return band_blocks(m, h) * kBandWaves * band_lists_of(v); }
__host__ __device__ inline int64_t band_max_bands(int64_t k, int v) { return (k + band_rows_of(v) - 1) / band_rows_of(v); }
__host__ __device__ inline int64_t band_head_stride(int64_t k, int v) { return band_max_bands(k, v) + 5; }
// The lists that workgroup w of a launch looks at for one that is heavy, where no launch before it could: all of them, or, of more than kBandTestAll, band_tests() from band_test_from() on, as far as
// there are any.  Then those that band_test_says() names have all of them together and say so, for the workgroups that begin later; a matrix with many heavy lists has one in any 256.
// (All of them by every workgroup are lists x lists: conversion with its count, us, the order by rows and the lists by launches of their own, all by every workgroup, and so; 32 rows per group, 2 %:
// 64000 x 1000, 2667 lists: 153 143 132; 128000 x 1000: 319 331 283; 400000 x 500, 5 %: 776 1375 648; 300000 x 128, 10 %: 418 784 368.  Power-law rows, 128000 x 1000: 238 301 237.  A single heavy
// list, the last one: 64000 x 1000 123 131 121.  From 1024 on for that: 32000 x 3000, 1334 lists, even 181 169 165, one heavy list 186 173 180; 24000 x 3000, 1000 lists, 256 of them by each were no faster, 121 to 119.)
constexpr int32_t kBandTestAll = 1024, kBandTestSome = 256;
__host__ __device__ inline int32_t band_tests(int32_t lists) { return lists <= kBandTestAll ? lists : kBandTestSome; }
__host__ __device__ inline int64_t band_test_from(int64_t w, int32_t lists) { return lists <= kBandTestAll ? 0 : w * kBandTestSome % lists; }
__host__ __device__ inline bool band_test_says(int64_t w, int32_t lists) { return lists <= kBandTestAll ? w == 0 : w * kBandTestSome < lists; }
// Entries of a (wave, band), on average, where the columns are uniform.
inline double band_entries(int64_t m, int64_t k, int64_t nnz, int32_t h, int v)
{
    const double blocks = (double)band_blocks(m, h), touched = (double)k * -std::expm1(-(double)nnz / blocks / (double)k);
    return (double)nnz / (blocks * kBandWaves) * band_rows_of(v) / (touched > 1.0 ? touched : 1.0);
}
// Upper bound of the units of all waves: a (wave, band) with n entries has at most n/4 + 2 steps, that is n/16 + 5/4 units and
// at least one.
__host__ __device__ inline int64_t band_units(int64_t nnz, int64_t m, int64_t k, int32_t h, int v)
{
    const int64_t lists = band_blocks(m, h) * kBandWaves * band_max_bands(k, v);
    return nnz / 16 + lists + (lists < nnz ? lists : nnz) + kBandSlackUnits;
}

}  // namespace gcoo
