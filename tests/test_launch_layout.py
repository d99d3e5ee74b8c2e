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
