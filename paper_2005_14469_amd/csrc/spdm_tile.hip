// The SpDM kernel that works row by row on a tile of B in LDS, and its launcher.
#include "gcoo_spdm_tile_kernel.hpp"

#include <atomic>

namespace gcoo {

hipError_t launch_spdm_rows_tile(const RowsArgs& a, int64_t row_wgs, bool whole, hipStream_t s)
{
    if (a.m < 1 || a.k < 1 || a.N < kTileCols || row_wgs < 1 || a.nnz > kTileMaxNnz || (uint64_t)a.k * (uint64_t)a.ldb * 4u > kRowsMaxBytes) return hipErrorInvalidValue;
    const int64_t tiles = (a.N + kTileCols - 1) / kTileCols, rows = (a.m + row_wgs - 1) / row_wgs, wgs = (a.m + rows - 1) / rows, total = tiles * wgs;
    const int64_t lds = tile_lds(a.k, rows);
    if (rows > kTileMaxRows || lds > kTileLdsBytes || total > 0x7ffffff0LL) return hipErrorInvalidValue;
    // more LDS than the default limit of a workgroup: asked for once per device
    static std::atomic<unsigned> done[64];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!done[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&spdm_rows_tile), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLdsBytes);
        if (e != hipSuccess) return e;
        done[dev].store(1u, std::memory_order_release);
    }
    // A row of three times the mean keeps its slot busy while the others of the wave have ended; rows of the open bin are not put in order among each other.
    const int64_t steps = (3 * (a.nnz / a.m) + 64) / 4;
    spdm_rows_tile<<<dim3((unsigned)((total + 7) / 8 * 8)), dim3(kTileThreads), (size_t)lds, s>>>(a, (int32_t)wgs, (int32_t)rows, (int32_t)total,
                                                                                                  (int32_t)(whole ? -1 : (steps < kTileBins - 2 ? steps : kTileBins - 2)));
    return hipGetLastError();
}

}  // namespace gcoo
