"""Enforcement at the largest model whose tile pairs the chip holds at once (31 blocks of 64 rows
on 256 CUs) and past it: an eager call against a captured one, which streams F through memory
once per iteration, bit for bit; alone and in batches with smaller models."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu, torch

pytestmark = pytest.mark.gpu


def _model(n, seed):
    rng = np.random.default_rng(seed + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    return dev(F), dev(rng.uniform(0.5, 2.0, n)), dev(rng.integers(100, 10000, n).astype(float))


def _captured(call):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    g.replay()
    torch.cuda.synchronize()


@pytest.mark.parametrize("n", [65, 1000, 1985, 2367, 2432, 2433, 2497])
def test_single(n):
    need_gpu()
    import paper_2511_04277_amd as rad
    F, area, rays = _model(n, 1)
    f1, f2 = F.clone(), F.clone()
    rad.enforce_vf_(f1, area, rays, tol=0.0, max_iter=6)
    _captured(lambda: rad.enforce_vf_(f2, area, rays, tol=0.0, max_iter=6, want_stats=False))
    assert torch.equal(f1, f2)


@pytest.mark.parametrize("sizes", [[2432], [2433], [2500, 1200], [2500, 2400, 2300, 100], [2400, 1000, 900, 64, 20]])
def test_batch(sizes):
    need_gpu()
    import paper_2511_04277_amd as rad
    models = []
    for k, n in enumerate(sizes):
        F, area, rays = _model(n, 10 + k)
        eps = dev(np.full(n, 0.5))
        models.append({"F": F, "area": area, "n_rays": rays, "eps": [eps], "rho": [1.0 - eps]})
    start = [m["F"].clone() for m in models]
    batch = rad.Batch(models, precision="fp64")
    batch.run(enforce_iters=6)
    got = [host(m["F"]) for m in models]
    for m, f in zip(models, start):
        m["F"].copy_(f)
    _captured(lambda: batch.run(enforce_iters=6))
    for a, m in zip(got, models):
        assert np.array_equal(a, host(m["F"]))
