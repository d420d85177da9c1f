// Workgroup -> output tile, shared by the matrix-product kernels.
#ifndef DYNB_TILE_MAP_H
#define DYNB_TILE_MAP_H

#include <hip/hip_runtime.h>

namespace dynb {

// Consecutive workgroup ids are spread round-robin over the 8 XCDs, each with its own L2: give
// every XCD a contiguous chunk of the tile sequence, and walk the tiles in bands of 8 tile-rows
// so that a chunk covers a compact rectangle (few distinct operand panels per L2).
__device__ inline void tile_of_block(int pid, int tiles_i, int tiles_j, int& ti, int& tj) {
  const int total = tiles_i * tiles_j;
  const int per = total / 8, extra = total % 8, xcd = pid % 8, local = pid / 8;
  int t = pid;
  if (total >= 16) t = xcd * per + (xcd < extra ? xcd : extra) + local;
  const int band = 8;
  const int bsz = band * tiles_j;
  const int b0 = t / bsz, r = t % bsz;
  const int rows = (tiles_i - b0 * band) < band ? (tiles_i - b0 * band) : band;
  ti = b0 * band + r % rows;
  tj = r / rows;
}

}  // namespace dynb

#endif
