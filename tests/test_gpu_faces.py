"""The CTU face kernels where their decomposition changes: tiles and marches (whole
grids of about 9 2^16 cells), march lengths (about 3 2^19 cells; group lists of few
and of many boxes), ragged rows, lines and tiles, occupancy maps built by one block
and by many.

Bars: FP64 against the oracle within 1e-12 of each component's largest value, FP32
within 1e-5 of it (of the flow's momentum scale for the momenta) wherever a float
rounding of the input moves the oracle's own result by less (flip_mask.py); listed groups bit-identical to the same cells of a whole-grid step, which the
arithmetic of both forms has in common.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from flip_mask import check_outside, sensitive_mask  # noqa: E402
from paper_1804_03479_amd import inputs  # noqa: E402
from paper_1804_03479_amd.mhd import Level, Solver  # noqa: E402

RECON = {"plm": oracle.PLM, "ppm": oracle.PPM}
SOLVERS = {"roe": oracle.ROE, "hlle": oracle.HLLE, "hlld": oracle.HLLD}


def level(U, B, dx, dtype=torch.float64, **kw):
    return Level(torch.from_numpy(U).to("cuda", dtype).contiguous(), torch.from_numpy(B).to("cuda", dtype).contiguous(),
                 dx, **kw)


@pytest.mark.parametrize("shape,recon,solver", [
    ((5, 4, 7), "ppm", "hlld"), ((67, 5, 4), "ppm", "roe"), ((4, 4, 131), "plm", "hlld"),
    ((41, 40, 39), "ppm", "hlld"), ((41, 40, 40), "ppm", "hlld"), ((41, 40, 40), "plm", "roe"),
    ((73, 73, 73), "ppm", "hlld"), ((74, 73, 73), "ppm", "hlld"), ((74, 73, 73), "ppm", "hlle"),
    ((84, 84, 83), "ppm", "hlld"), ((84, 84, 83), "plm", "roe"), ((84, 84, 84), "ppm", "hlld"),
    ((117, 116, 116), "ppm", "hlld")])
def test_whole_grid_step(shape, recon, solver):
    p = inputs.smooth_problem(*shape, seed=sum(shape))
    U, B = oracle.initial_state(p)
    dt = oracle.cfl_dt(U, B, p["dx"])
    Uo, Bo = oracle.step(U, B, dt, p["dx"], scheme=oracle.CTU, recon=RECON[recon], riemann=SOLVERS[solver])
    s, lv = Solver("ctu", recon, solver), level(U, B, p["dx"])
    s.step(lv, dt)
    for got, want in ((lv.U, Uo), (lv.B, Bo)):
        got = got.cpu().numpy()
        for m in range(len(want)):
            assert np.abs(got[m] - want[m]).max() <= 1e-12 * np.abs(want[m]).max()


@pytest.mark.parametrize("shape,recon,solver", [
    ((5, 6, 4), "ppm", "hlld"), ((17, 20, 30), "ppm", "hlld"), ((31, 32, 33), "ppm", "hlld"), ((32, 32, 32), "ppm", "hlld"),
    ((84, 84, 83), "ppm", "hlld"), ((84, 84, 84), "ppm", "hlld"), ((33, 32, 31), "plm", "hlle"),
    ((69, 69, 68), "plm", "roe"), ((69, 69, 69), "plm", "roe")])
def test_whole_grid_step_f32(shape, recon, solver):
    p = inputs.smooth_problem(*shape, seed=sum(shape))
    U, B = (a.astype(np.float32).astype(np.float64) for a in oracle.initial_state(p))
    dt = oracle.cfl_dt(U, B, p["dx"])

    def run(u, b):
        return oracle.step(u, b, dt, p["dx"], scheme=oracle.CTU, recon=RECON[recon], riemann=SOLVERS[solver])

    s, lv = Solver("ctu", recon, solver, "f32"), level(U, B, p["dx"], torch.float32)
    s.step(lv, dt)
    check_outside(lv.U.double().cpu().numpy(), lv.B.double().cpu().numpy(), *run(U, B), *sensitive_mask(run, U, B),
                  max_frac=1e-3, what=f"{shape} {recon} {solver}")


@pytest.mark.parametrize("edge,n,groups,prec", [(16, 128, 1, "f32"), (16, 128, 40, "f64"), (16, 128, 300, "f32"),
                                                (4, 100, 9, "f64"), (4, 104, 9, "f32")])
def test_listed_groups_equal_whole_grid(edge, n, groups, prec):
    dtype = torch.float64 if prec == "f64" else torch.float32
    U, B = oracle.initial_state(p := inputs.smooth_problem(n, n, n, seed=4))
    m = n // edge
    pick = np.random.default_rng(groups).choice(m ** 3, groups, replace=False)
    origins = np.stack([pick % m, pick // m % m, pick // m ** 2], 1) * edge
    s = Solver("ctu", "ppm", "hlld", prec)
    whole = level(U, B, p["dx"], dtype)
    part = level(U, B, p["dx"], dtype, groups=torch.from_numpy(origins.astype(np.int32)).cuda(), group_edge=edge)
    U0, B0 = part.U.clone(), part.B.clone()
    dt = s.cfl_dt(whole)
    s.step(whole, dt)
    s.step(part, dt)
    cell = torch.zeros((n, n, n), dtype=torch.bool, device="cuda")
    for i, j, k in origins:
        cell[k:k + edge, j:j + edge, i:i + edge] = True
    assert torch.equal(part.U, torch.where(cell, whole.U, U0))
    for a in range(3):                     # a listed cell's faces, its upper ones included
        face = cell | torch.roll(cell, 1, 2 - a)
        assert torch.equal(part.B[a], torch.where(face, whole.B[a], B0[a]))


@pytest.mark.parametrize("shape,recon,solver", [((5, 4, 7), "plm", "roe"), ((48, 48, 48), "plm", "roe"),
                                                ((32, 40, 100), "ppm", "hlld"), ((32, 40, 103), "ppm", "hlld")])
def test_vl_whole_grid_step(shape, recon, solver):
    # the VL flux stage split by direction (fewer than 512 blocks of 256 cells) and whole
    p = inputs.smooth_problem(*shape, seed=sum(shape))
    U, B = oracle.initial_state(p)
    dt = oracle.cfl_dt(U, B, p["dx"])
    Uo, Bo = oracle.step(U, B, dt, p["dx"], scheme=oracle.VL, recon=RECON[recon], riemann=SOLVERS[solver])
    s, lv = Solver("vl", recon, solver), level(U, B, p["dx"])
    s.step(lv, dt)
    for got, want in ((lv.U, Uo), (lv.B, Bo)):
        got = got.cpu().numpy()
        for m in range(len(want)):
            assert np.abs(got[m] - want[m]).max() <= 1e-12 * np.abs(want[m]).max()
