"""Interface capture of a CTU step: which faces a stride samples and what is recorded.

Bars: the number of records exactly; every record of a strided capture one of the records
of the full capture of the same step, bit for bit; the recorded flux the solver's on the
recorded states within 2e-5 (FP32 rounding), as in test_gpu_mlp.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_1804_03479_amd import inputs  # noqa: E402
from paper_1804_03479_amd.mhd import Level, MlpOps, Solver  # noqa: E402


def records(solver, U, B, dx, stride, groups=None, edge=16):
    s = Solver("ctu", "ppm", solver, "f32")
    ops = MlpOps(s)
    lv = Level(torch.from_numpy(U).to("cuda", torch.float32), torch.from_numpy(B).to("cuda", torch.float32), dx,
               groups=groups, group_edge=edge)
    buf = torch.zeros((2 * 3 * lv.U[0].numel() * 2, 22), dtype=torch.float32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    ops.set_capture(buf, count, stride)
    s.step(lv, oracle.cfl_dt(U, B, dx))
    ops.set_capture(None)
    torch.cuda.synchronize()
    n = int(count.item())
    return n, buf[:n].cpu().numpy()


@pytest.mark.parametrize("shape", [(4, 5, 6), (17, 9, 13), (40, 24, 31)])
@pytest.mark.parametrize("solver", ["hlld", "hlle"])
@pytest.mark.parametrize("stride", [2, 3, 7, 96, 100003])
def test_strided_records_of_a_whole_grid(shape, solver, stride):
    p = inputs.smooth_problem(*reversed(shape), seed=sum(shape))
    U, B = oracle.initial_state(p)
    faces = 3 * int(np.prod(shape))
    n, every = records(solver, U, B, p["dx"], 1)
    assert n == 2 * faces                  # both Riemann stages
    n, some = records(solver, U, B, p["dx"], stride)
    assert n == 2 * ((faces - 1) // stride + 1)
    full = {r.tobytes() for r in every}
    assert all(r.tobytes() in full for r in some)
    for r in some[:: max(1, n // 40)].astype(np.float64):
        f, _ = oracle.riemann({"hlld": oracle.HLLD, "hlle": oracle.HLLE}[solver], r[:7], r[7:14], r[14])
        assert np.allclose(r[15:], f, rtol=2e-5, atol=2e-5 * np.abs(f).max())


def test_strided_records_of_listed_groups():
    p = inputs.smooth_problem(32, 32, 32, seed=9)
    U, B = oracle.initial_state(p)
    g = torch.tensor([(16, 0, 0), (0, 16, 16)], dtype=torch.int32, device="cuda")
    n, every = records("hlld", U, B, p["dx"], 1, groups=g)
    full = {r.tobytes() for r in every}
    for stride in (3, 50):
        m, some = records("hlld", U, B, p["dx"], stride, groups=g)
        assert 0 < m < n and all(r.tobytes() in full for r in some)
