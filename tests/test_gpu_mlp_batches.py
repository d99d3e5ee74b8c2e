"""Batches of the network's kernels at the edges of their tiling: 16 rows to a
wave, 64 to a block, at most 1024 blocks (inference) or 256 (gradients), so a
second tile per block begins past 65,536 and 16,384 rows.

Bars as in test_gpu_mlp.py, element by element: both sides round the same
operands to BF16, and an activation that the FP32 accumulation order moves
across a rounding boundary moves an output by one BF16 ulp of one term.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import mlp as omlp  # noqa: E402
from paper_1804_03479_amd.mhd import MlpOps, Solver  # noqa: E402

RTOL, ATOL = 1e-2, 2e-3


def close(a, b, what):
    a = a.double().cpu().numpy()
    bound = RTOL * np.abs(b) + ATOL * np.abs(b).max()
    assert (np.abs(a - b) <= bound).all(), (what, float((np.abs(a - b) / bound).max()))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("n", [1, 15, 17, 63, 64, 65, 16384, 16385, 65537 + 64])
def test_rows_at_tile_edges(n):
    rng = np.random.default_rng(n)
    th = (omlp.init_params(3) + 0.05 * rng.standard_normal(omlp.NPARAM)).astype(np.float32).astype(np.float64)
    X = rng.standard_normal((n, 15)).astype(np.float32).astype(np.float64)
    dY = rng.standard_normal((n, 7)).astype(np.float32).astype(np.float64)
    ops = MlpOps(Solver("ctu", "ppm", "mlp", "f32"))
    Yo, cache = omlp.forward(th, X, bf16_ops=True)
    close(ops.forward(dev(th), dev(X)), Yo, "forward")
    G = ops.backward(dev(th), dev(X), dev(dY))
    Go = omlp.backward(th, cache, dY, bf16_ops=True)
    for k, (a, b) in enumerate(zip(omlp.unpack(G.double().cpu().numpy()), omlp.unpack(Go))):
        close(torch.from_numpy(np.asarray(a)), b, f"gradient part {k}")
    # the training step's own gradient and loss, and the same bits on a second run
    runs = []
    for _ in range(2):
        p, m, v, g = dev(th), dev(0 * th), dev(0 * th), dev(0 * th)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        ops.train_step(p, m, v, g, 1, dev(X), dev(dY), 1e-3, loss)
        runs.append(torch.cat([p, m, v, g, loss]))
    assert torch.equal(*runs)
    lo, go = omlp.mse_grad(th, X, dY, bf16_ops=True)
    assert abs(loss.item() - lo) <= 1e-3 * lo
    close(g, go, "training gradient")
