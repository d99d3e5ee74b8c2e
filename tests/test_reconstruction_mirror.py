"""The reconstruction's exact symmetry: mirrored cells give mirrored edge values, bit for
bit, in both precisions.  csrc/mhd_device.hpp compiled for the CPU, no GPU."""

import pytest

from test_launch_layout import run_host

PRELUDE = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
static inline float rsqrtf(float x) { return 1.0f / std::sqrt(x); }
static inline double rsqrt(double x) { return 1.0 / std::sqrt(x); }
#define __builtin_amdgcn_fmed3f(a, b, c) fmaxf(fminf(a, b), fminf(fmaxf(a, b), c))
#include "mhd_device.hpp"
using namespace mhd;
#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } } while (0)
"""


@pytest.mark.parametrize("real", ["float", "double"])
def test_ppm_edges_of_mirrored_cells(tmp_path, real):
    run_host(tmp_path, r"""
typedef %s real;
int main() {
  std::mt19937 rng(7);
  std::normal_distribution<double> g;
  for (int n = 0; n < 200000; ++n) {
    real q[5], l, r, ml, mr;
    for (int c = 0; c < 5; ++c) q[c] = real(n %% 3 == 0 ? g(rng) : n %% 3 == 1 ? std::exp(2 * g(rng)) : 1 + 0.1 * c + 0.01 * g(rng));
    ppm_edges(q[0], q[1], q[2], q[3], q[4], l, r);
    ppm_edges(q[4], q[3], q[2], q[1], q[0], ml, mr);
    CHECK(l == mr && r == ml, "cells %%.17g %%.17g %%.17g %%.17g %%.17g: %%.17g %%.17g, mirrored %%.17g %%.17g", (double)q[0],
          (double)q[1], (double)q[2], (double)q[3], (double)q[4], (double)l, (double)r, (double)mr, (double)ml);
    // and of the negative ones
    ppm_edges(-q[0], -q[1], -q[2], -q[3], -q[4], ml, mr);
    CHECK(l == -ml && r == -mr, "negative cells");
  }
}""" % real, prelude=PRELUDE)
