// Where the dense pass reads X: address and range of the buffer load of one 16 x 16 tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nnr {

// The "row" orientation of one tile: lane (l16, row) holds X[i0 + l16][j0 + 4*row + r], r = 0..3, one 16-byte raw buffer
// load per lane.  The buffer starts at the strip's first row and the panel's first column (wave-uniform) and ends where the
// tensor ends.  The hardware compares every dword's offset FROM VOFFSET ALONE with that range and returns zero for what lies
// beyond; a scalar offset (soffset) is added to the address but not to what is compared, so a load has none: the tile
// column is part of the lane's offset.  A tile beyond the matrix, or a strip's rows beyond the last slice, may then be asked
// for without a branch.
struct TileBuffer {
  int64_t first;                                    // element of X that the buffer starts at
  uint32_t bytes;                                   // its range (what lies 4 GB behind the start is never asked for)
};
__host__ __device__ inline TileBuffer tile_buffer(int64_t n, int64_t total, int t, int64_t i0, int64_t jp0) {
  const int64_t first = (t * n + i0) * n + jp0, bytes = 4 * (total - first);
  return TileBuffer{first, (uint32_t)(bytes < 0xFFFFFFFFLL ? bytes : 0xFFFFFFFFLL)};
}
__host__ __device__ inline uint32_t tile_lane_offset(uint32_t n, int l16, int row) { return ((uint32_t)l16 * n + 4u * row) * 4u; }
__host__ __device__ inline uint32_t tile_voffset(uint32_t lane_offset, int jt) { return lane_offset + 64u * (uint32_t)jt; }

}  // namespace nnr
