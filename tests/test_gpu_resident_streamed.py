"""The on-chip enforcement bitwise against the streamed one, which a captured run takes: every size
class, both forms of kappa, the tolerance stop with its statistics, and every iteration count over two
rounds of the buffers that are used in turn (two and four iterations)."""
import numpy as np
import pytest

from tests.gpu_util import dev, need_gpu, padded, torch

pytestmark = pytest.mark.gpu

KEYS = ("iters", "converged", "closure_defect", "recip_err", "device_status")


def _compare(n, kappa, tol, iters):
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    area, rays = dev(rng.uniform(0.5, 2.0, n)), dev(rng.integers(100, 10000, n).astype(float))
    half = dev(np.full(n, 0.5))
    start, f = dev(F), dev(F)
    batch = rad.Batch([{"F": f, "area": area, "n_rays": rays, "eps": [half], "rho": [half]}], precision="fp64",
                      kappa=kappa)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        batch.run(enforce_iters=iters, enforce_tol=tol)
    g.replay()
    want, streamed = batch.stats()[0], f.clone()
    f.copy_(start)
    batch.run(enforce_iters=iters, enforce_tol=tol)
    got = batch.stats()[0]
    assert torch.equal(f, streamed)
    assert [got[k] for k in KEYS] == [want[k] for k in KEYS]
    f1 = padded(F, n + 9)
    st = rad.enforce_vf_(f1, area, rays, kappa=kappa, tol=tol, max_iter=iters)
    assert torch.equal(f1, streamed)
    assert [st[k] for k in KEYS] == [want[k] for k in KEYS]
    return want


@pytest.mark.parametrize("kappa", ["fracvar", "half"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 700, 1408, 1409, 1984, 1985])
def test_tolerance_stop(n, kappa):
    need_gpu()
    _compare(n, kappa, 1e-3, 12)


@pytest.mark.parametrize("n,iters", [(130, k) for k in range(1, 10)] + [(1450, k) for k in range(2, 10)] +
                         [(64, 333), (65, 333), (700, 64), (1984, 40)])
def test_iteration_counts(n, iters):
    need_gpu()
    assert _compare(n, "fracvar", 0.0, iters)["iters"] == iters
