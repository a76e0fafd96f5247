// The sixteen-wave SpDM kernel that reads the band schedule, and its launcher.
#include "gcoo_spdm_band_kernel.hpp"

#include <atomic>

namespace gcoo {

template <int V, bool SPREAD, bool LATE>
static hipError_t launch_band(const BandArgs& a, const RowsArgs& rows, const BandRowsGrid& rg, hipStream_t s)
{
    // more LDS than the default limit of a workgroup: asked for once per device
    static std::atomic<unsigned> done[64];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!done[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&spdm_band<V, SPREAD, LATE>), hipFuncAttributeMaxDynamicSharedMemorySize, kBandLdsBytes);
        if (e != hipSuccess) return e;
        done[dev].store(1u, std::memory_order_release);
    }
    spdm_band<V, SPREAD, LATE><<<dim3((unsigned)(a.grid > kRowsAllWgs ? a.grid : kRowsAllWgs)), dim3(64 * kBandWaves), kBandLdsBytes, s>>>(a, rows, rg);
    return hipGetLastError();
}

hipError_t launch_spdm_band(const BandArgs& a, const RowsArgs& rows, hipStream_t s)
{
    if (a.v != 2 && a.v != 4) return hipErrorInvalidValue;
    const int64_t tile = 64 * a.v, tiles = (a.N + tile - 1) / tile, total = a.blocks * tiles;
    if (total <= 0 || total > 0x7ffffff0LL) return hipErrorInvalidConfiguration;
    if (a.h < 1 || a.h > 96 / a.v || a.blocks != band_blocks(a.m, a.h) || a.head_stride != band_head_stride(a.k, a.v)) return hipErrorInvalidValue;
    if ((uint64_t)a.k * (uint64_t)a.ldb * 4u > kRowsMaxBytes) return hipErrorInvalidValue;
    const bool aligned = a.N % 4 == 0 && a.ldb % 4 == 0 && reinterpret_cast<uintptr_t>(a.B) % 16 == 0;
    if (a.v == 2 && a.k > kBandTallMaxK) return hipErrorInvalidValue;
    if (!aligned && a.N < tile) return hipErrorInvalidValue;
    BandArgs b = a;
    b.total = (int32_t)total;
    b.grid = (int32_t)((total + 7) / 8 * 8);                 // whole rounds over the 8 XCDs
    BandRowsGrid rg;
    const int64_t mean = rows.nnz / rows.m, wave_row = 2 * mean > 64 ? 2 * mean : 64;
    if (rows.N < 4) return hipErrorInvalidConfiguration;
    RowsArgs by_rows = rows;
    by_rows.moved = rows_moved(rows.m, rows.nnz, rows.N, rows.C, rows.ldc);
    rg.tiles = (int32_t)((rows.N + by_rows.moved + 63) / 64);
    rg.rpw = 4;                                              // (8: as fast)
    rg.wave_row = (int32_t)(wave_row > INT32_MAX ? INT32_MAX : wave_row);
    // How the rows of B are requested goes by the entries of a (wave, band).  Product alone, against behind the first unit, mean of 20 to 200 matrices each; wide:
    //   entries                    8 - 10  12 - 14  14 - 16  17 - 18  19 - 20  20 - 21  22 - 23  25 - 26  28 - 29  36 - 40  40 - 50  80 - 150
    //   a row at a time             0.975    0.978    0.993    1.025    1.028    1.038    1.043    1.043    1.051    1.043    1.044     1.021
    //   behind the second step      0.999    0.985    0.986    0.993    0.998    1.002    1.007    1.010    1.016    1.012    1.013     1.006
    //   behind the second unit      1.000    1.018    1.031    1.088    1.095    1.105    1.089    1.062    1.047    1.007    0.998     0.997
    // tall:
    //   entries                   14 - 16  16 - 18  18 - 20  20 - 22  24 - 26  28 - 32  32 - 36  36 - 40  40 - 50   60 - 80
    //   a row at a time             0.989    0.990    0.997    1.003    1.029    1.049    1.052    1.056    1.056     1.055
    //   behind the second step      1.004    1.006    1.009    1.010    1.014    1.027    1.033    1.033    1.031     1.024
    //   behind the second unit      0.996    0.994    1.006    1.018    1.022    1.019    1.009    0.996    0.986     0.973
    const double entries = band_entries(a.m, a.k, rows.nnz, a.h, a.v);
    if (a.v == 2) {
        if (entries < 20.0) return launch_band<2, true, false>(b, by_rows, rg, s);
        return entries < 37.0 ? launch_band<2, false, false>(b, by_rows, rg, s) : launch_band<2, false, true>(b, by_rows, rg, s);
    }
    if (entries < 20.0) return entries < 14.0 ? launch_band<4, true, false>(b, by_rows, rg, s) : launch_band<4, true, true>(b, by_rows, rg, s);
    return entries < 42.0 ? launch_band<4, false, false>(b, by_rows, rg, s) : launch_band<4, false, true>(b, by_rows, rg, s);
}

}  // namespace gcoo
