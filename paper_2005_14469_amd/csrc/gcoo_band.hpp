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
