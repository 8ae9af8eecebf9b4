// spin_tile.h -- what the kernels that run several sweeps of a tile in LDS share
// (k_block, k_heis_block): which tile a workgroup takes and the order of the
// rows of its region.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spin {

// Workgroups are dealt to the 8 XCDs round-robin: give each XCD a contiguous run of tiles, whose
// shared halos then come from one L2.  A permutation of 0 .. gridDim.x - 1 for any grid.
__device__ __forceinline__ uint32_t xcd_tile() {
  const uint32_t n = gridDim.x, q = n >> 3, r = n & 7u, xcd = blockIdx.x & 7u;
  return xcd * q + (xcd < r ? xcd : r) + (blockIdx.x >> 3);
}

// Place of region row (y, z) of Y x Z (2D: Z = 1, z = 0) in a list of the rows from the innermost
// outwards: the rows at least s away from the region's edge are its first (Y - 2s)(Z - 2s) entries
// (2D: Y - 2s), so a colour phase that may only update those takes the front of the list.
template <int D>
__device__ __forceinline__ uint32_t tile_row_rank(uint32_t y, uint32_t z, uint32_t Y, uint32_t Z) {
  uint32_t s = y < Y - 1u - y ? y : Y - 1u - y;  // shell: distance from the edge
  if (D == 2) {
    const uint32_t ny = Y - 2u * s;
    return (ny > 2u ? ny - 2u : 0u) + (y == s ? 0u : 1u);
  }
  const uint32_t sz = z < Z - 1u - z ? z : Z - 1u - z;
  s = s < sz ? s : sz;
  const uint32_t ny = Y - 2u * s, nz = Z - 2u * s;
  const uint32_t inner = (ny > 2u ? ny - 2u : 0u) * (nz > 2u ? nz - 2u : 0u);
  if (z == s) return inner + (y - s);
  if (z == Z - 1u - s) return inner + ny + (y - s);
  if (y == s) return inner + 2u * ny + (z - s - 1u);
  return inner + 2u * ny + (nz - 2u) + (z - s - 1u);
}

// Rows at least s away from the edge of a Y x Z region.
template <int D>
__device__ __forceinline__ uint32_t tile_rows(uint32_t Y, uint32_t Z, uint32_t s) {
  return D == 3 ? (Y - 2u * s) * (Z - 2u * s) : Y - 2u * s;
}

}  // namespace spin
