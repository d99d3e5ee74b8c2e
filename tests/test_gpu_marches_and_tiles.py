"""The face kernels' forms against each other, bit for bit, on ragged grids: a grid below
the switch between tiles and marches, and the same periodic state repeated until it is
above.  A face's arithmetic is the same in both, so the repeated grid's step is the small
one's repeated -- for the learned flux too, whose network runs on a wave's 64 faces
whichever they are.  And the learned flux of marches on the faces themselves: a strided
capture's count, and its fluxes against the reference surrogate on the recorded states
(element by element, the bars of test_gpu_mlp.py)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from oracle import mlp as omlp  # noqa: E402
from paper_1804_03479_amd import inputs  # noqa: E402
from paper_1804_03479_amd.mhd import Level, MlpOps, Solver  # noqa: E402

TILE_LIMIT = 9 << 16


def theta():
    th = omlp.init_params(3) + 0.05 * np.random.default_rng(1).standard_normal(omlp.NPARAM)
    return th.astype(np.float32).astype(np.float64)


def solver_of(riemann, prec, recon="ppm"):
    s = Solver("ctu", recon, riemann, prec)
    if riemann == "mlp":
        MlpOps(s).set_weights(torch.from_numpy(theta().astype(np.float32)).cuda())
    return s


# (small grid, repeats along z, y, x)
CASES = [((17, 84, 83), (5, 1, 1)), ((85, 42, 83), (1, 2, 1)), ((85, 84, 28), (1, 1, 3)), ((5, 200, 300), (2, 1, 1)),
         ((45, 53, 21), (1, 1, 12))]


@pytest.mark.parametrize("small,times", CASES)
@pytest.mark.parametrize("riemann,prec,recon", [("mlp", "f32", "ppm"), ("mlp", "f32", "plm"), ("hlld", "f32", "ppm"),
                                                ("hlld", "f64", "ppm"), ("roe", "f32", "plm"), ("roe", "f64", "ppm")])
def test_marches_repeat_the_tiles(small, times, riemann, prec, recon):
    n = int(np.prod(small))
    assert n < TILE_LIMIT <= n * int(np.prod(times))
    p = inputs.smooth_problem(*reversed(small), seed=sum(small))
    U, B = oracle.initial_state(p)
    dt = oracle.cfl_dt(U, B, p["dx"])
    dtype = torch.float32 if prec == "f32" else torch.float64
    U, B = torch.from_numpy(U).to("cuda", dtype), torch.from_numpy(B).to("cuda", dtype)
    a, b = Level(U.clone(), B.clone(), p["dx"]), Level(U.repeat(1, *times), B.repeat(1, *times), p["dx"])
    s = solver_of(riemann, prec, recon)
    for _ in range(2):
        s.step(a, dt)
        s.step(b, dt)
    assert torch.isfinite(a.U).all()
    assert torch.equal(b.U, a.U.repeat(1, *times)) and torch.equal(b.B, a.B.repeat(1, *times))


# group lists on both sides of the switches (item boxes of 20^3 and 18^3 cells for groups
# of 16^3: 2^20 cells of them for 16 columns, 2^22 for 8; large boxes 9 2^16), in one launch
# and in batches, the list's length on the host and on the device
@pytest.mark.parametrize("edge,side,groups,riemann,prec", [
    (16, 128, 131, "hlld", "f32"), (16, 128, 132, "hlld", "f32"), (16, 128, 179, "hlle", "f32"), (16, 128, 180, "hlle", "f32"),
    (16, 144, 524, "hlld", "f64"), (16, 144, 525, "roe", "f32"), (16, 144, 719, "mlp", "f32"), (16, 144, 720, "mlp", "f32"),
    (8, 64, 37, "roe", "f64"), (4, 52, 300, "mlp", "f32"), (32, 96, 12, "roe", "f64"), (32, 96, 13, "roe", "f64"),
    (32, 96, 13, "hlld", "f32"), (48, 96, 4, "hlld", "f64"), (48, 96, 5, "hlld", "f64")])
def test_lists_of_tiles_and_of_marches_equal_the_whole_grid(edge, side, groups, riemann, prec):
    p = inputs.smooth_problem(side, side, side, seed=groups)
    U, B = oracle.initial_state(p)
    dtype = torch.float32 if prec == "f32" else torch.float64
    U, B = torch.from_numpy(U).to("cuda", dtype), torch.from_numpy(B).to("cuda", dtype)
    m = side // edge
    pick = np.random.default_rng(groups).choice(m ** 3, groups, replace=False)
    origins = (np.stack([pick % m, pick // m % m, pick // m ** 2], 1) * edge).astype(np.int32)
    s = solver_of(riemann, prec)
    whole = Level(U.clone(), B.clone(), p["dx"])
    dt = 0.7 * s.cfl_dt(whole)
    s.step(whole, dt)
    for batch, used in ((0, None), (groups // 3 + 1, None), (0, max(1, groups - 3))):
        s.set_launch(0, 0, batch)
        part = Level(U.clone(), B.clone(), p["dx"], groups=torch.from_numpy(origins).cuda(), group_edge=edge)
        if used is not None:
            part.n_groups_dev = torch.tensor([used], dtype=torch.int32, device="cuda")
        s.step(part, dt)
        cell = torch.zeros((side,) * 3, dtype=torch.bool, device="cuda")
        for i, j, k in origins[:used]:
            cell[k:k + edge, j:j + edge, i:i + edge] = True
        assert torch.equal(part.U, torch.where(cell, whole.U, U))
        for a in range(3):
            face = cell | torch.roll(cell, 1, 2 - a)
            assert torch.equal(part.B[a], torch.where(face, whole.B[a], B[a]))


@pytest.mark.parametrize("shape,stride", [((85, 84, 83), 197), ((85, 84, 83), 4098), ((5, 347, 353), 1001)])
def test_learned_flux_of_marched_faces(shape, stride):
    n = int(np.prod(shape))
    assert n >= TILE_LIMIT
    p = inputs.abc_problem(96, 0.1, seed=4)
    U, B = oracle.initial_state(p)
    reps = [-(-s // 96) for s in shape]
    U, B = (np.tile(q, [1] + reps)[:, :shape[0], :shape[1], :shape[2]] for q in (U, B))   # jumps at the seams: HLLD there
    lv = Level(torch.from_numpy(U.astype(np.float32)).cuda(), torch.from_numpy(B.astype(np.float32)).cuda(), p["dx"])
    s = solver_of("mlp", "f32")
    ops = MlpOps(s)
    faces = 2 * ((3 * n - 1) // stride + 1)
    buf = torch.zeros((faces + 64, 22), dtype=torch.float32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    ops.set_capture(buf, count, stride)
    s.step(lv, 0.5 * s.cfl_dt(lv))
    ops.set_capture(None)
    torch.cuda.synchronize()
    assert int(count.item()) == faces
    S = buf[:faces].double().cpu().numpy()
    wl, wr, bn, F = S[:, :7], S[:, 7:14], S[:, 14], S[:, 15:]
    fall = omlp.fallback(wl, wr)
    assert (~fall).sum() > faces // 2
    Fo = omlp.surrogate_flux(theta(), wl[~fall], wr[~fall], bn[~fall], bf16_ops=True)
    bound = 1e-2 * np.abs(Fo) + 2e-3 * np.abs(Fo).max()
    assert (np.abs(F[~fall] - Fo) <= bound).all()
    for i in np.flatnonzero(fall)[:40]:
        fo, _ = oracle.riemann(oracle.HLLD, wl[i], wr[i], bn[i])
        assert np.allclose(F[i], fo, rtol=2e-5, atol=2e-5 * np.abs(fo).max())
