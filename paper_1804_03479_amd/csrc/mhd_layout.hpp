// mhd_layout.hpp -- index arithmetic that decides which cell a thread reads and
// which blocks cover a level.  No kernel and no launch in here: a host compiler
// takes it as well, so its bounds can be gone through on the CPU for every size.
#pragma once
#include <hip/hip_runtime.h>

namespace mhd {

// n / d for 0 <= n < 2^31 by a divisor fixed on the host (make_div): one high
// multiply, an add and a shift instead of a division's reciprocal sequence.
struct FastDiv {
  unsigned m, a, s;
};
__host__ __device__ __forceinline__ unsigned fdiv(const FastDiv& f, unsigned n) {
  return ((unsigned)(((unsigned long long)n * f.m) >> 32) + (n & f.a)) >> f.s;
}
// d = 1: n itself.  d > 1: s = ceil(log2 d) - 1, m = floor(2^(32 + s) / d) + 1
// < 2^32; m d exceeds 2^(32 + s) by at most d <= 2^(s + 1), so the quotient is
// exact for n < 2^31.
inline FastDiv make_div(unsigned d) {
  if (d <= 1) return FastDiv{0u, ~0u, 0u};
  unsigned s = 0;
  while ((2ull << s) < d) ++s;
  return FastDiv{(unsigned)((1ull << (32 + s)) / d + 1), 0u, s};
}

struct Work {
  int nx, ny, nz;
  long long N;          // cells of the grid
  const int* groups;    // nullptr: whole grid
  int edge;             // group edge in cells
  int halo;             // extra cells around each group
  int box;              // edge + 2 * halo
  long long items;      // work items (cells), upper bound when n_dev is set
  const int* occ;       // group occupancy map (list mode), gnx*gny*gnz
  int gnx, gny, gnz;    // groups per dimension
  const int* n_dev;     // list mode: number of groups read from device memory, or nullptr
  int gbase;            // list mode: first group of this launch (a batch of the list)
  int gcount;           // list mode: groups of this launch at most
  int oshift;           // list mode: group origins are divided by 2^oshift (coarse footprint)
  // Stage scratch (W, F, E, Q, Bh, ...) addressing.  Whole grid: like the
  // level (slot = cell index, stride N).  Group list: each group owns a
  // contiguous box of sb^3 slots (its cells plus sb/2 - edge/2 ghost layers),
  // group g at slot (g + 1) sb^3, with one unused box before and after so
  // stencil reads past a box edge stay inside the allocation.
  long long NS;         // component stride of the scratch arrays
  int sb;               // scratch box edge (0: scratch addressed like the level)
  int soff;             // offset of this stage's item box inside the scratch box
  // Block decomposition of the stage kernels (Cell): units (the grid's
  // z-planes, the listed groups' item boxes, or the grid as one row of cells) of
  // `per` cells, each covered by `chunks` blocks.
  int units;
  unsigned per, chunks;
  int rev;              // walk the blocks from the last to the first
  FastDiv by_chunks, by_row, by_plane;   // of the block rank; of a cell index by its row and by its plane
  FastDiv by_box;       // of an item index by a group's item box (cell_of)
  FastDiv by_edge;      // of a cell coordinate by the group edge
};

// How a stage kernel's threads find their cells (Cell): the z-planes of a whole grid,
// the item boxes of a group list, or a whole grid's cells one after the other.
constexpr int kWhole = 0, kList = 1, kFlat = 2;

// The planes form has its plane's address in scalar registers, but a plane fills whole
// blocks: 4 x 4 cells use 16 of 256 lanes.  The flat form wraps along z per thread and
// fills every lane; it is taken where planes fill less than 9/10 of their blocks, if a
// component's bytes fit its 32-bit offsets.  Whole step (us), planes / flat, VL + PLM +
// Roe float and double, 16 of 256 lanes: 65536 x 4 x 4 (z first) 960 / 226 by stages;
// 1/4: 4096 x 8 x 8 104 / 70 and 208 / 119; 0.53: 4096 x 16 x 17 303 / 206 and 756 / 484;
// 0.78: 1000 x 24 x 25 134 / 126 and 270 / 241; 0.83: 600 x 32 x 33 135 / 127 and 278 /
// 244; 0.98: 300 x 50 x 50 145 / 147 and 312 / 299; 1: 4096 x 16 x 16 192 / 193 and 449 /
// 450, 128^3 404 / 415 and 955 / 938.
inline bool flat_pays(long long nx, long long ny, long long nz, int elem, int threads) {
  const long long plane = nx * ny, lanes = (plane + threads - 1) / threads * threads;
  return nx * ny * nz * elem <= 0xffffffffLL && 10 * plane < 9 * lanes;
}

// Block decomposition of a stage kernel for blocks of `threads`: fills the Work's unit
// fields and returns the number of blocks
inline long long decompose(Work& w, int mode, int threads) {
  if (w.groups) {
    w.per = (unsigned)(w.box * w.box * w.box);
    w.units = (int)(w.items / w.per);
    w.by_row = make_div((unsigned)w.box);
    w.by_plane = make_div((unsigned)(w.box * w.box));
  } else if (mode == kFlat) {
    w.per = (unsigned)w.N;
    w.units = 1;
    w.by_row = make_div((unsigned)w.nx);
    w.by_plane = make_div((unsigned)w.nx * (unsigned)w.ny);
  } else {
    w.per = (unsigned)((long long)w.nx * w.ny);
    w.units = w.nz;
    w.by_row = make_div((unsigned)w.nx);
  }
  w.chunks = (w.per + (unsigned)threads - 1) / (unsigned)threads;
  w.by_chunks = make_div(w.chunks);
  return (long long)w.units * w.chunks;
}

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
