"""The index arithmetic of the kernels (csrc/mhd_layout.hpp), gone through on the CPU
for whole ranges of sizes: compiled with the host compiler, no GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1804_03479_amd", "csrc")

PRELUDE = r"""
#include <cstdio>
#include <cstdlib>
#include "mhd_layout.hpp"
using namespace mhd;
#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } } while (0)
"""


def run_host(tmp_path, body, prelude=PRELUDE):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(prelude + body)
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                          str(src), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout


@pytest.mark.parametrize("tile", [16, 8, 4])
def test_staged_tile_coordinates_stay_in_the_grid(tmp_path, tile):
    # every column a block of k_emf_tiled stages is a cell of the grid, and the ones
    # its cells use are the periodic ones
    run_host(tmp_path, r"""
int main() {
  for (int n = 4; n <= 200; ++n)
    for (int t0 = 0; t0 < n; t0 += %d)
      for (int h = 0; h <= %d; ++h) {
        const int x = staged_coord(t0, h, n);
        CHECK(x >= 0 && x < n, "n %%d tile at %%d column %%d: reads %%d", n, t0, h, x);
        if (t0 - 1 + h < n) CHECK(x == (t0 - 1 + h + n) %% n, "n %%d tile at %%d column %%d: %%d", n, t0, h, x);
      }
}""" % (tile, tile))


def test_stage_blocks_fill_their_lanes(tmp_path):
    # whole grids, in the form the step picks: at least three quarters of the lanes
    # launched have a cell wherever the grid itself fills a few blocks
    run_host(tmp_path, r"""
int main() {
  const int sizes[] = {4, 5, 6, 7, 8, 9, 12, 16, 17, 24, 33, 61, 64, 97, 128, 200, 512, 4096, 65536};
  for (int threads = 64; threads <= 512; threads += 64)
    for (int nx : sizes) for (int ny : sizes) for (int nz : sizes) {
      const long long n = (long long)nx * ny * nz;
      if (n > 1LL << 28 || n < 8 * threads) continue;
      Work w{};
      w.nx = nx; w.ny = ny; w.nz = nz; w.N = w.items = n;
      const int mode = flat_pays(nx, ny, nz, 4, threads) ? kFlat : kWhole;
      const long long lanes = decompose(w, mode, threads) * threads;
      CHECK(lanes >= n && 3 * lanes <= 4 * n, "%d x %d x %d, blocks of %d: %lld lanes for %lld cells", nx, ny, nz, threads, lanes, n);
    }
}""")


def test_cells_of_the_flat_form(tmp_path):
    # the splitting of a cell number by multiplications, for every cell of odd grids and
    # for the last cells of the largest component 32-bit offsets reach
    run_host(tmp_path, r"""
static void check(int nx, int ny, int nz, unsigned from) {
  Work w{};
  w.nx = nx; w.ny = ny; w.nz = nz; w.N = w.items = (long long)nx * ny * nz;
  decompose(w, kFlat, 256);
  CHECK(w.per == (unsigned)w.N && w.units == 1 && w.chunks == (w.N + 255) / 256, "decomposition");
  for (unsigned l = from; l < w.per; ++l) {
    const unsigned k = fdiv(w.by_plane, l), r = l - k * (unsigned)nx * (unsigned)ny, j = fdiv(w.by_row, r);
    CHECK(k == l / ((unsigned)nx * ny) && j == r / (unsigned)nx, "%d x %d x %d cell %u", nx, ny, nz, l);
  }
}
int main() {
  for (int nx = 4; nx < 40; nx += 3) for (int ny = 4; ny < 40; ny += 5) check(nx, ny, 41, 0);
  check(4, 4, 1 << 26, (1u << 30) - 100000);
  check(5, 7, ((1 << 30) - 1) / 35, 35u * (((1u << 30) - 1) / 35) - 100000);
  check(1 << 13, 1 << 13, 16, (1u << 30) - 100000);
}""")


@pytest.mark.parametrize("cols", [8, 16])
def test_face_slabs_of_whole_grids(tmp_path, cols):
    # the slabs cover the grid once; no wave task traces many lanes per face; and no slab
    # of a large grid holds more cells than its three directions can share in a cache
    run_host(tmp_path, r"""
int main() {
  const int sizes[] = {4, 5, 6, 7, 8, 9, 12, 16, 17, 24, 33, 61, 64, 97, 128, 200, 400, 512, 1024, 4096, 65536};
  for (int nx : sizes) for (int ny : sizes) for (int nz : sizes) {
    const long long n = (long long)nx * ny * nz;
    if (n > 1LL << 28 || n < 1 << 14) continue;
    Work w{};
    w.nx = nx; w.ny = ny; w.nz = nz; w.N = w.items = n;
    const FaceGeo g = face_geometry(w, %d);
    const long long sz = g.slabs / (g.ux * g.uy);
    CHECK(g.units == g.slabs && sz * g.ux * g.uy == g.slabs, "%%d x %%d x %%d: units", nx, ny, nz);
    CHECK(sz * g.bz >= nz && (sz - 1) * g.bz < nz && (long long)g.uy * g.by >= ny && (g.uy - 1LL) * g.by < ny &&
          (long long)g.ux * g.bx >= nx && (g.ux - 1LL) * g.bx < nx,
          "%%d x %%d x %%d: %%d slabs of %%d x %%d x %%d", nx, ny, nz, (int)g.units, g.bx, g.by, g.bz);
    CHECK(g.units * g.per < 1LL << 31, "waves");
    long long traced = 0;                  // waves' traces; marches trace one cell more than they have
    for (int k0 = 0; k0 < nz; k0 += g.bz) for (int j0 = 0; j0 < ny; j0 += g.by) {
      const int bz = nz - k0 < g.bz ? nz - k0 : g.bz, by = ny - j0 < g.by ? ny - j0 : g.by;
      long long per = (long long)g.per - g.w2 - g.w1;
      if (g.tz) per += g.w2 + g.w1;
      else per += ((long long)g.bx * by + 63) / 64 * (bz + (bz + g.cz - 1) / g.cz) +
                  ((long long)g.bx * bz + 63) / 64 * (by + (by + g.cy - 1) / g.cy);
      traced += per * g.ux;
    }
    traced *= 64;
    // (planes of 20 cells leave 12 of 32 columns of a pair of tiles empty)
    CHECK(traced <= 3 * n * (nx * ny < kTilePlane || nx * nz < 64 ? 10 : 7) / 4, "%%d x %%d x %%d: %%lld lanes trace %%lld faces", nx, ny, nz, traced, 3 * n);
    CHECK(n < 1 << 20 || nx * nz < 64 || 4LL * g.bx * g.by * g.bz <= n, "%%d x %%d x %%d: slabs of %%d x %%d x %%d", nx, ny, nz, g.bx, g.by, g.bz);
  }
}""" % cols)


def test_division_by_a_fixed_divisor(tmp_path):
    # every divisor at the multiples around which a quotient could round, up to 2^31 - 1
    run_host(tmp_path, r"""
static void check(unsigned d) {
  const FastDiv f = make_div(d);
  for (int e = 0; e < 32; ++e)
    for (long long q = -2; q <= 2; ++q)
      for (long long o = -1; o <= 1; ++o) {
        const long long n = ((1LL << e) / d + q) * d + o;
        if (n >= 0 && n < 1LL << 31) CHECK(fdiv(f, (unsigned)n) == (unsigned)n / d, "%lld / %u", n, d);
      }
  const unsigned last = (1u << 31) - 1;
  for (unsigned n : {last, last - last % d, last - last % d - 1}) CHECK(fdiv(f, n) == n / d, "%u / %u", n, d);
}
int main() {
  for (unsigned d = 1; d < 200000; ++d) check(d);
  for (unsigned d = 200000; d < 1u << 31; d += d / 1000 + 7) check(d);
  for (int b = 1; b < 31; ++b) for (int o = -1; o <= 1; ++o) check((1u << b) + o);
}""")


def test_flux_grid_keeps_the_block_limit(tmp_path):
    # a launch row per direction only for levels of little work, whatever the limit, and
    # never more blocks than the limit (of at least three: one a row)
    run_host(tmp_path, r"""
int main() {
  const int cu = 256;
  for (long long blocks = 1; blocks < 100000; blocks += 1 + blocks / 7)
    for (int per_cu = 0; per_cu <= 16; ++per_cu) {
      const FluxGrid g = flux_blocks(blocks, cu, (long long)per_cu * cu);
      CHECK(g.y == (blocks < 2 * cu ? 3u : 1u), "%lld blocks of work, %d per CU: %u rows", blocks, per_cu, g.y);
      CHECK(per_cu == 0 ? g.x == blocks : (long long)g.x * g.y <= (long long)per_cu * cu && g.x <= blocks,
            "%lld blocks of work, %d per CU: %u x %u", blocks, per_cu, g.x, g.y);
    }
}""")


def test_largest_grid_of_the_face_kernels(tmp_path):
    # every byte offset of the largest component is below 2^32; the next grid is refused
    run_host(tmp_path, r"""
int main() {
  for (int elem : {4, 8}) {
    const long long most = (1LL << 32) / elem - 1;
    CHECK(face_addressable(most, elem) && (most - 1) * elem <= 0xffffffffLL, "%d bytes", elem);
    CHECK(!face_addressable(most + 1, elem), "%d bytes: a component of 4 GiB", elem);
    CHECK(98 * (most + 1) * elem > 288LL << 30, "the budget of a refused grid");
  }
}""")


def test_blocks_of_the_largest_levels(tmp_path):
    # the diagnostics' blocks cover every level that is accepted (up to 2^34 cells, planes
    # of up to 2^32) with numbers of cells in a unit and of blocks that fit their words
    run_host(tmp_path, r"""
int main() {
  for (int elem : {4, 8})
    for (int ax = 2; ax <= 32; ++ax) for (int ay = 2; ax + ay <= 32; ++ay) for (int d = 0; d < 2; ++d) {
      const long long nx = (1LL << ax) - (ax > 2 ? d : 0), ny = 1LL << ay;
      if (nx > 1LL << 30 || ny > 1LL << 30) continue;
      long long nz = (1LL << 34) / (nx * ny);
      if (nz > 1 << 30) nz = 1 << 30;
      Work w{};
      w.nx = (int)nx; w.ny = (int)ny; w.nz = (int)nz; w.N = w.items = nx * ny * nz;
      const long long blocks = decompose(w, read_mode(w, elem), 256);
      CHECK(blocks < 1LL << 31 && (long long)w.units * w.per >= w.N && (w.units - 1LL) * w.per < w.N && w.chunks * 256LL >= w.per,
            "%lld x %lld x %lld: %d units of %u cells, %lld blocks", nx, ny, nz, w.units, w.per, blocks);
      for (long long limit : {0LL, 256LL, 1LL << 40})
        CHECK(launch_blocks(blocks, limit) * (long long)kMaxBlock < 1LL << 32 && launch_blocks(blocks, limit) <= blocks,
              "%lld x %lld x %lld: launch of %u blocks", nx, ny, nz, launch_blocks(blocks, limit));
    }
}""")


@pytest.mark.parametrize("cols", [8, 16])
def test_face_slabs_of_group_lists(tmp_path, cols):
    # every group's box whole, in tiles whose waves share one cell or in slabs of marches
    run_host(tmp_path, r"""
int main() {
  const int cols = %d;
  static int origin[3];
  for (int box = 6; box <= 140; ++box)
    for (long long groups = 1; groups < 3000; groups += 1 + groups / 3) {
      Work w{};
      w.groups = origin; w.box = box; w.nx = w.ny = w.nz = 4096; w.N = 1LL << 36;
      w.items = groups * box * box * box;
      const FaceGeo g = face_geometry(w, cols);
      const long long sz = g.slabs;
      CHECK(g.ux == 1 && g.uy == 1 && g.bx == box && g.by == box && g.lx == box && g.units == groups * sz, "%%d: slabs", box);
      CHECK(sz * g.bz >= box && (sz - 1) * g.bz < box, "box %%d: %%lld slabs of %%d planes", box, sz, g.bz);
      if (g.tz) {
        const long long cells = 64 / cols, waves = ((long long)g.tz * box - 1 + cells - 2) / (cells - 1);
        CHECK(sz == 1 && g.tz == g.ty && (long long)g.tz * cols >= box * box && g.w2 == waves && g.w1 == waves &&
              (long long)waves * (cells - 1) + 1 >= (long long)g.tz * box, "box %%d: tiles", box);
      } else {
        // as many cells as a slab may have, in whole marches
        CHECK(sz == 1 || (long long)box * box * (g.bz - g.cz) <= kListSlab, "box %%d: slab of %%d planes", box, g.bz);
      }
      CHECK(g.units * g.per < 1LL << 31, "waves");
    }
}""" % cols)
