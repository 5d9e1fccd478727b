// Which tile of a tiled launch a block has (gemm.hip, mxfp4.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace paro {

constexpr int kBandTiles = 8;                       // token tiles of a band that is walked output tile by output tile

// Blocks are numbered so that 32 neighbours on one XCD (block id mod 8) form a patch of 8 (token tiles) x 4 (output tiles) that
// walks K in step and shares activation and weight panels through that XCD's L2: tiles are counted in bands of 8 token tiles,
// output tile by output tile, dealt to the XCDs 32 at a time, and what does not fill a round of 256 in eight equal runs, so
// that every XCD has the same number of tiles to one.  A launch has `all` tiles rounded up to 8 as blocks; false: none left.
__device__ __forceinline__ bool tile_index(int all, int &idx)
{
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, j_rest = all / 256 * 32;          // of this XCD; the first of its run
    idx = j < j_rest ? (j / 32 * 8 + xcd) * 32 + j % 32 : j_rest * 8 + xcd * ((int)(gridDim.x >> 3) - j_rest) + j - j_rest;
    return idx < all;
}

__device__ __forceinline__ void tile_place(int tile, int m_tiles, int n_tiles, int &m, int &n)
{
    const int whole = m_tiles / kBandTiles * kBandTiles * n_tiles;                         // tiles of whole bands
    const int high = tile < whole ? kBandTiles : m_tiles % kBandTiles, first = tile < whole ? 0 : whole;
    const int column = (tile - first) / high, m_band = tile < whole ? column / n_tiles * kBandTiles : m_tiles - high;
    m = m_band + (tile - first) % high;
    n = column % n_tiles;
}

}  // namespace paro
