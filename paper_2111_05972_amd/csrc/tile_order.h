// Which output tile a workgroup of a GEMM launch computes, shared by the bf16 and the float kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace tpl {

// Workgroup id -> position in the tile list.  Consecutive ids go to different XCDs (each with its
// own L2), so ids are regrouped to give every XCD one contiguous run of the list.
__device__ __forceinline__ int share_of_block(int bid, int nblocks) {
    constexpr int NXCD = 8;
    int per = nblocks / NXCD, rem = nblocks % NXCD;
    int xcd = bid % NXCD, idx = bid / NXCD;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}
// Tile order: column-major inside bands of `band` tile rows.  Every XCD (own L2) works through one contiguous run
// of this list (share_of_block), i.e. a block of band rows x some columns of the tile grid: it fetches the A panels
// of its band and the B panels of its columns once.  The host picks the band height that minimises the sum over
// XCDs of those fetches (choose_band).
__device__ __forceinline__ void tile_coords(int tile, int tiles_m, int tiles_n, int band_rows, int& tm, int& tn) {
    int band_tiles = band_rows * tiles_n;
    int band = tile / band_tiles, within = tile % band_tiles;
    int rows = tiles_m - band * band_rows;
    rows = rows < band_rows ? rows : band_rows;
    tm = band * band_rows + within % rows;
    tn = within / rows;
}

}  // namespace tpl
