"""Diagnostics and CFL step against the FP64 oracle at the edges of their
decomposition: planes below, at and above one block of 256 cells, more blocks
than one residency, listed groups, and a level whose planes pass 4 GiB.

Bars: sums of n terms in another order differ by at most n epsilon of the sum of
the terms' magnitudes, here taken 100 times smaller (the reductions are trees);
the divergence is compared per cell, so its maximum is exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_1804_03479_amd import inputs  # noqa: E402
from paper_1804_03479_amd.mhd import Level, Solver  # noqa: E402


def totals(U, B, dx):
    up = [np.roll(B[a], -1, 2 - a) for a in range(3)]
    c = [0.5 * (B[a] + up[a]) for a in range(3)]
    q = [U[m] for m in range(5)] + [0.5 * (c[0] ** 2 + c[1] ** 2 + c[2] ** 2),
                                    0.5 * (U[1] ** 2 + U[2] ** 2 + U[3] ** 2) / U[0]]
    div = sum((up[a] - B[a]) * (1.0 / dx) for a in range(3))
    return q, div


@pytest.mark.parametrize("prec,nx,ny,nz", [("f64", 4, 5, 6), ("f32", 16, 16, 5), ("f64", 257, 1, 4), ("f32", 61, 97, 130),
                                           ("f64", 128, 96, 160)])
def test_totals_and_divergence(prec, nx, ny, nz):
    ny = max(ny, 4)
    dtype = torch.float32 if prec == "f32" else torch.float64
    p = inputs.smooth_problem(nx, ny, nz, seed=nx)
    U, B = oracle.initial_state(p)
    rng = np.random.default_rng(nx)
    B = B + 0.01 * rng.standard_normal(B.shape)          # a divergence above rounding
    U, B = (torch.from_numpy(a).to("cuda", dtype) for a in (U, B))
    s, lv = Solver("ctu", "ppm", "hlld", prec), Level(U.contiguous(), B.contiguous(), p["dx"])
    U, B = U.double().cpu().numpy(), B.double().cpu().numpy()
    q, div = totals(U, B, p["dx"])
    for got, v in zip(s.sums(lv), q):
        assert abs(got - v.sum() * p["dx"] ** 3) <= 1e-2 * v.size * 2.3e-16 * np.abs(v).sum() * p["dx"] ** 3 + 1e-14
    mx, l1 = s.divb(lv)
    assert abs(mx - np.abs(div).max()) <= 1e-15 * np.abs(B).max() / p["dx"]
    assert abs(l1 - np.abs(div).mean()) <= 1e-15 * np.abs(B).max() / p["dx"]
    assert abs(s.cfl_dt(lv) / oracle.cfl_dt(U, B, p["dx"]) - 1.0) <= (1e-5 if prec == "f32" else 1e-13)


def test_listed_groups_only():
    p = inputs.smooth_problem(48, 32, 32, seed=2)
    U, B = oracle.initial_state(p)
    g = torch.tensor([[32, 16, 0], [0, 0, 16]], dtype=torch.int32, device="cuda")
    lv = Level(torch.from_numpy(U).cuda(), torch.from_numpy(B).cuda(), p["dx"], groups=g)
    q, _ = totals(U, B, p["dx"])
    for got, v in zip(Solver().sums(lv), q):
        want = (v[0:16, 16:32, 32:48].sum() + v[16:32, 0:16, 0:16].sum()) * p["dx"] ** 3
        assert abs(got - want) <= 1e-12 * np.abs(v).sum() * p["dx"] ** 3


def test_planes_beyond_4_gib():
    nz, ny, nx = 4, 16384, 32769
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free device memory")
    U = torch.zeros((5, nz, ny, nx), dtype=torch.float64, device="cuda")
    B = torch.zeros((3, nz, ny, nx), dtype=torch.float64, device="cuda")
    U[0] = 1.0
    U[4] = 1.5
    U[1, 3, ny - 1, nx - 1] = 2.0        # the last cell moves: v^2 / 2 = 2, its pressure stays 1
    U[4, 3, ny - 1, nx - 1] = 3.5
    B[0, 3, ny - 1, 0] = 0.25            # its upper x face, across the wrap
    s, lv = Solver("vl", "plm", "hlld", "f64"), Level(U, B, 1.0)
    n = float(nx) * ny * nz
    t = s.sums(lv)
    assert t[0] == n and t[1] == 2.0 and abs(t[4] - (1.5 * n + 2.0)) <= 1e-12 * n
    assert t[5] == 2 * 0.5 * 0.125 ** 2 and t[6] == 2.0
    assert s.divb(lv) == (0.25, 0.5 / n)
    a = 5.0 / 3.0 * (1.0 - 0.5 * 0.125 ** 2 * 2.0 / 3.0)   # sound speed squared with the face's field in the cell
    fast = np.sqrt(a + 0.125 ** 2)
    small = 0.5 / (2.0 + fast + 2 * fast)
    assert abs(s.cfl_dt(lv) / small - 1.0) < 0.05
