// The band schedule: the kernel-private listing that the sixteen-wave SpDM kernel reads (gcoo_spdm_band_kernel.hpp).
//
// A block is kBandWaves x h consecutive rows of A, wave w of the workgroup owning rows [w*h, (w+1)*h) of it (h <= 24; the
// blocks have nothing to do with the groups of the format).  The distinct columns of a block, ascending, are cut into bands
// of 80: the rows of B that are in LDS together, band b in buffer b mod 2.
//
// Units.  The entries of one (wave, band) are listed in steps of four records, four steps to a unit of 128 bytes, which
// the kernel fetches into scalar registers.  A record is 8 bytes:
//     { value (fp32 bits), row inside the wave's rows | place of its B row in LDS << 10 }     place = (b mod 2) * 80 + slot
// The steps of a (wave, band) begin on a unit of their own.  First the pair steps: two pairs of entries of one column each
// (the second entry of a pair reuses the B values of the first, the reuse of Algorithm 2), then the single steps.
// Records without an entry hold value 0 and row kBandSink: they add zero into a partial sum that is never stored.  Every (wave,
// band) has at least one unit, so that the units of a wave follow each other without gaps.
//
// Order.  Columns ascend inside the pairs and inside the singles, rows ascend inside a column; the last row of a column
// with an odd count is the single.  A wave whose rows repeat a coordinate has singles only, in row order.
//
// Heads.  head[(block * 16 + w) * stride + i], i = 0 .. bands + 1, stride = band_head_stride(k): eight words
//     { the five columns whose B rows wave w fetches for band i; pair steps, single steps of band i - 1; unused }
// (bands beyond the last repeat the last column).  count[block] = distinct columns; first[block * 16 + w] = first unit of a wave.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gcoo {

constexpr int kBandWaves = 16;
constexpr int kBandRows = 80;            // rows of B per band, five per wave
constexpr int kBandMaxH = 24;            // rows of A per wave: (24 + 1) x 4 partial sums per lane in v[28:127]
constexpr int kBandSink = kBandMaxH;
constexpr int kBandHeadWords = 8;
constexpr int kBandUnitWords = 32;       // 16 records
constexpr int kBandSlackUnits = 2;       // read-ahead behind the last unit
constexpr int64_t kBandMaxK = 262144;    // the column bitmaps of a block are held in LDS

// A list of more entries than this makes the matrix an uneven one, for which no schedule is built: the sixteen waves wait for each other
// in every band, so a list of three times the mean has the others wait two thirds of the time.  Uniform lists stay far below (960
// entries +- 31 at 8000 x 8000, 0.5 %).
inline int32_t band_heavy(int64_t nnz, int64_t lists)
{
    const int64_t n = lists > 0 ? 3 * (nnz / lists) + 512 : 0;
    return (int32_t)(n > INT32_MAX ? INT32_MAX : n);
}
__host__ __device__ inline int64_t band_blocks(int64_t m, int32_t h) { return (m + kBandWaves * h - 1) / (kBandWaves * h); }
__host__ __device__ inline int64_t band_max_bands(int64_t k) { return (k + kBandRows - 1) / kBandRows; }
__host__ __device__ inline int64_t band_head_stride(int64_t k) { return band_max_bands(k) + 5; }
// Upper bound of the units of all waves: a (wave, band) with n entries has at most n/4 + 2 steps, that is n/16 + 5/4 units and
// at least one.
__host__ __device__ inline int64_t band_units(int64_t nnz, int64_t m, int64_t k, int32_t h)
{
    const int64_t lists = band_blocks(m, h) * kBandWaves * band_max_bands(k);
    return nnz / 16 + lists + (lists < nnz ? lists : nnz) + kBandSlackUnits;
}

}  // namespace gcoo
