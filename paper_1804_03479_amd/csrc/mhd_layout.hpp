// mhd_layout.hpp -- index arithmetic that decides which cell a thread reads and
// which blocks cover a level.  No kernel and no launch in here: a host compiler
// takes it as well, so its bounds can be gone through on the CPU for every size.
#pragma once
#include <hip/hip_runtime.h>

namespace mhd {

// a coordinate at most one period outside 0..n-1, wrapped into it
__host__ __device__ __forceinline__ int wrapc(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Coordinate h of a staged tile (h = 0: the layer below the tile's first cell t0) on
// an axis of n cells: the layer wraps, columns past the grid, which no cell reads,
// repeat its last one.  wrapc() would take a tile that is longer than the grid out
// of its range (n < 8 with 16 cells along x).
__host__ __device__ __forceinline__ int staged_coord(int t0, int h, int n) {
  const int i = t0 - 1 + h;
  return i < 0 ? i + n : (i < n ? i : n - 1);
}

}  // namespace mhd
