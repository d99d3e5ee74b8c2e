// mhd_layout.hpp -- index arithmetic that decides which cell a thread reads and
// which blocks cover a level.  No kernel and no launch in here: a host compiler
// takes it as well, so its bounds can be gone through on the CPU for every size.
#pragma once
#include <hip/hip_runtime.h>

namespace mhd {

// n / d for 0 <= n < 2^31 by a divisor fixed on the host (make_div): a shift, one high
// multiply and a shift instead of a division's reciprocal sequence.
struct FastDiv {
  unsigned m, s;
};
__host__ __device__ __forceinline__ unsigned fdiv(const FastDiv& f, unsigned n) {
  return (unsigned)(((unsigned long long)(2u * n) * f.m) >> 32) >> f.s;
}
// s = ceil(log2 d), m = floor(2^(31 + s) / d) + 1 < 2^32; m d exceeds 2^(31 + s) by at
// most d <= 2^s, so the quotient is exact for n < 2^31.
inline FastDiv make_div(unsigned d) {
  if (d <= 1) return FastDiv{(1u << 31) + 1u, 0u};
  const unsigned s = 32u - (unsigned)__builtin_clz(d - 1);
  return FastDiv{(unsigned)((1ull << (31 + s)) / d + 1), s};
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

// The kernels that only read the level (CFL, diagnostics) address it by 64-bit indices in a
// group list, and where a plane of a whole grid passes 4 GiB (kList without a list).
inline int read_mode(const Work& w, int elem) {
  return w.groups || (long long)w.nx * w.ny * elem > 0xffffffffLL ? kList : kWhole;
}

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
  } else if (mode == kList) {
    w.per = 1u << 30;   // planes may have 2^32 cells
    w.units = (int)((w.N + w.per - 1) / w.per);
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

// Blocks of a launch over `blocks` blocks of work, at most max_blocks (0: no limit of the
// caller's).  A launch has fewer than 2^32 threads; a kernel's blocks walk the rest.
constexpr int kMaxBlock = 512;   // largest block of the step's stage kernels (tuned per context)
constexpr long long kMaxLaunch = 0xffffffffLL / kMaxBlock;
inline unsigned launch_blocks(long long blocks, long long max_blocks) {
  if (max_blocks > 0 && blocks > max_blocks) blocks = max_blocks;
  if (blocks > kMaxLaunch) blocks = kMaxLaunch;
  return (unsigned)(blocks < 1 ? 1 : blocks);
}

// Grid of the VL flux stage for `blocks` blocks of work, at most max_blocks of them (0: no
// limit): where there are fewer than two blocks per CU, a launch row for each direction,
// as one wave's chain of loads and divisions is what they wait for.  The limit counts
// all rows and does not make a large level a small one.  Whole step (us), all directions
// in a thread / one each, VL + PLM + Roe: float 16^3 39 / 33, 32^3 41 / 36, 48^3 55 / 53,
// 64^3 66 / 70; double 32^3 57 / 48, 40^3 74 / 66, 48^3 74 / 75, 64^3 122 / 125
struct FluxGrid {
  unsigned x, y;
};
inline FluxGrid flux_blocks(long long blocks, int num_cu, long long max_blocks) {
  const unsigned rows = blocks < 2LL * num_cu ? 3 : 1;
  const long long limit = max_blocks / rows;
  return FluxGrid{launch_blocks(blocks, max_blocks > 0 && limit < 1 ? 1 : limit), rows};
}

// Decomposition of the CTU face kernels (k_ctu_faces): slabs of rows and planes of a
// whole grid or of a group's item box, each cut into wave tasks.
struct FaceGeo {
  int bx, by, bz;          // cells of a slab
  int ux, uy;              // slabs side by side along x and y
  unsigned slabs;          // of a box (of the grid)
  long long units;         // slabs of the launch
  int cz, cy;              // cells of a z-march and of a y-march
  int lx;                  // positions of a row in the x-rows: one more than its cells on a periodic grid
  unsigned w2, w2c;        // waves of a slab's z-marches, and of one chunk of them
  unsigned w1, w1c;        // ... y-marches
  unsigned per;            // waves of a slab
  FastDiv by_per, by_slabs, by_ux, by_uy, by_w2c, by_w1c, by_bx, by_by, by_lx;
  unsigned tz, ty;         // z and y in tiles: tiles side by side (0: in marches)
  FastDiv by_ly, by_lz;
};

// The face kernels address a component of a whole grid by 32-bit byte offsets.  A grid of
// components of 4 GiB and more is refused as out of memory, without a look at what the
// device holds: its step is budgeted at 98 words a cell (mhd_workspace_bytes), 392 GiB
// at that size, more than a gfx950 device has, and was always refused so.
inline bool face_addressable(long long cells, int elem) { return cells * elem < 1LL << 32; }

// A march repeats the trace of one cell before its first face, so long marches save
// work and short ones give small grids enough waves.
//
// Whole grids below kTileLimit cells go in tiles of `cols` columns: they trace less per
// face than short marches, which read along whole rows.  Whole step (us), marches /
// tiles, CTU + PPM + HLLD unless stated: double 24^3 53 / 44, 48^3 101 / 82, 64^3 172 /
// 147, 80^3 289 / 268, 96^3 486 / 509; float 24^3 35 / 34, 48^3 54 / 49, 80^3 130 / 119,
// 96^3 188 / 186, 128^3 464 / 525; float Roe (PLM) 64^3 107 / 98, 80^3 179 / 165, 96^3
// 249 / 260; learned flux 32^3 57 / 51, 64^3 172 / 159, 128^3 1021 / 1079.
// So do grids whose planes are less than two waves of z-marches, or where not even all
// planes fill the lanes of a y-march (65536 x 4 x 4, z first,
// double 998 / 646; 65536 x 8 x 8 2776 / 2603; 4096 x 16 x 17 667 / 681).
//
// A slab's three directions read the same cells one after the other: a slab as large as
// the grid leaves the caches in between.  CTU + PPM + HLLD (Roe), double, with slabs of
// a march's planes only / as below: 4 x 512 x 512 881 / 590 (1353 / 831), 8 x 512 x 512
// 2314 / 1164 (3743 / 1635), 4 x 1024 x 1024 5458 / 2344 (8794 / 3285), 8 x 8 x 65536
// 4778 / 2319 (7683 / 3300); tiles of 65536 x 4 x 4 680 / 646, of 20000 x 10 x 10 1339 /
// 1232; lists of one box of 64^3 270 / 218 (391 / 295), of 128^3 3056 / 1477.
constexpr long long kTileLimit = 9 << 16;
constexpr long long kTilePlane = 128;
constexpr long long kTileSlab = 1 << 16;   // cells
constexpr long long kListSlab = 1 << 15;
// Lists go in tiles as well, up to these many cells in all item boxes: for 8 and for 16
// columns, and for boxes of more than kListSlab cells (kTileLimit).  Whole step (us),
// marches / tiles, 16^3 groups, CTU + PPM: HLLD float 1 / 8 / 30 / 150 / 300 groups 38 /
// 35, 52 / 47, 98 / 89, 361 / 361, 709 / 729; double 4 / 30 / 300 / 511 / 1024 64 / 53, 177
// / 149, 1545 / 1491, 2596 / 2607, 5167 / 5248; Roe double 8 / 100 / 511 103 / 81, 712 /
// 632, 3422 / 3285; learned flux 100 / 511 469 / 417, 2203 / 2084; boxes: 4 of 48^3 HLLD
// double 376 / 352, 10 of them 881 / 917, 2 of 32^3 Roe double 139 / 100.
constexpr long long kTileList8 = 4 << 20;
constexpr long long kTileList16 = 1 << 20;

inline FaceGeo face_geometry(const Work& w, int cols) {
  FaceGeo g;
  g.tz = g.ty = 0;
  g.ux = g.uy = 1;
  const auto cut = [](long long n, long long len) { return (int)((n + len - 1) / len); };
  const bool list = w.groups != nullptr;
  const int nx = list ? w.box : w.nx, ny = list ? w.box : w.ny, nz = list ? w.box : w.nz;
  const long long plane = (long long)nx * ny, boxes = list ? w.items / (plane * nz) : 1;
  // lists: whole float step of 5 / 50 / 191 / 400 groups: 54 / 152 / 531 / 1098 us
  // with marches of 2 cells, 64 / 152 / 504 / 1029 with 5, 80 / 167 / 510 / 1017 with 10;
  // 1 / 4 / 8 groups in double 54 / 65 / 80 with 1, 63 / 70 / 81 with 2.
  // Whole grids, CTU + PPM + HLLD, marches of 2 / 4 / 8 cells: float 128^3 500 / 476 /
  // 474; double 96^3 515 / 490 / 514
  const long long n = w.items < 1 << 16 ? 1 : 2 + (w.items >> 18);
  const int len = list ? (n > 10 ? 10 : (int)n) : w.N < 3 << 19 ? 4 : 8;
  g.bx = nx;
  g.by = ny;
  g.bz = nz;
  g.cz = g.cy = len;
  if (list && w.items < (plane * nz > kListSlab ? kTileLimit : cols > 8 ? kTileList16 : kTileList8)) {
    g.tz = g.ty = (unsigned)cut(plane, cols);
    g.by_ly = g.by_lz = make_div((unsigned)nx);
  } else if (list) {
    const int parts = cut(plane * nz, kListSlab);
    if (parts > 1) g.bz = len * cut(nz, (long long)len * parts);
    if (g.bz > nz) g.bz = nz;
  } else if (w.N < kTileLimit || plane < kTilePlane || (long long)nx * nz < 64) {
    if (plane < kTilePlane && w.N >= 2 * kTileSlab) g.bz = (int)(kTileSlab / plane);
    g.tz = (unsigned)cut(plane, cols);
    g.ty = (unsigned)cut((long long)nx * g.bz, cols);
    g.by_ly = make_div((unsigned)ny + 1);
    g.by_lz = make_div((unsigned)g.bz + 1);
  } else {
    // planes of a march's length, of grids of few planes in equal parts; of several
    // marches where rows are short, so that the lanes of the y-marches (a row times the
    // planes) are four fifths in use
    if (nz < 4 * len) g.cz = cut(nz, nz < len ? 1 : (nz + len / 2) / len);
    g.bz = g.cz;
    while (g.bz < 8 * g.cz && 5LL * nx * g.bz < 4 * 64LL * cut((long long)nx * g.bz, 64)) g.bz *= 2;
    const int parts = nz < g.bz ? 1 : (nz + g.bz / 2) / g.bz;   // alike
    g.bz = g.cz * cut(nz, (long long)g.cz * parts);
    if (g.bz > nz) g.bz = nz;
    // where that leaves fewer than 16 slabs, parts of the planes and, last, of the rows
    const int sz = cut(nz, g.bz);
    if (sz < 16) g.by = len * cut(ny, (long long)len * cut(16, sz));
    if (g.by > ny) g.by = ny;
    g.uy = cut(ny, g.by);
    if (sz * g.uy < 16) g.bx = 64 * cut(nx, 64LL * cut(16, (long long)sz * g.uy));
    if (g.bx > nx) g.bx = nx;
    g.ux = cut(nx, g.bx);
  }
  g.lx = list ? nx : g.bx + 1;
  g.slabs = (unsigned)(g.ux * g.uy * cut(nz, g.bz));
  g.units = boxes * g.slabs;
  const auto waves = [](long long n, int k) { return (unsigned)((n + k - 1) / k); };
  g.w2c = waves((long long)g.bx * g.by, 64);
  g.w2 = g.w2c * (unsigned)cut(g.bz, g.cz);
  g.w1c = waves((long long)g.bx * g.bz, 64);
  g.w1 = g.w1c * (unsigned)cut(g.by, g.cy);
  if (g.tz) {
    g.w2 = waves((long long)g.tz * (g.bz + !list) - 1, 64 / cols - 1);
    g.w1 = waves((long long)g.ty * (g.by + !list) - 1, 64 / cols - 1);
  }
  g.per = g.w2 + g.w1 + waves((long long)g.lx * g.by * g.bz - 1, 63);
  g.by_per = make_div(g.per);
  g.by_slabs = make_div(g.slabs);
  g.by_ux = make_div((unsigned)g.ux);
  g.by_uy = make_div((unsigned)g.uy);
  g.by_w2c = make_div(g.w2c);
  g.by_w1c = make_div(g.w1c);
  g.by_bx = make_div((unsigned)g.bx);
  g.by_by = make_div((unsigned)g.by);
  g.by_lx = make_div((unsigned)g.lx);
  return g;
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
