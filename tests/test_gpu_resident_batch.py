"""A batch's models that fit the chip together run all enforcement iterations in one launch; a
captured run streams all of them, one launch per step.  Both give the same bits, for groups of
several models, more models than one group holds, models too large for one, and a bad model."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu, torch

pytestmark = pytest.mark.gpu


def _models(sizes):
    out = []
    for k, n in enumerate(sizes):
        rng = np.random.default_rng(97 * k + n)
        F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
        F[:, n] += 0.01
        F /= F.sum(axis=1, keepdims=True)
        eps = dev(rng.uniform(0.1, 0.9, n))
        out.append({"F": dev(F), "area": dev(rng.uniform(0.5, 2.0, n)),
                    "n_rays": dev(rng.integers(100, 10000, n).astype(float)), "eps": [eps], "rho": [1.0 - eps]})
    return out


@pytest.mark.parametrize("sizes", [[1, 40, 64], [65, 200, 700, 1], [1900, 1300, 900, 300, 30], [2100, 1500],
                                   [2100, 100, 200], [2050]])
@pytest.mark.parametrize("tol", [0.0, 1e-3])
def test_equals_captured_run(sizes, tol):
    need_gpu()
    import paper_2511_04277_amd as rad
    models = _models(sizes)
    start = [m["F"].clone() for m in models]
    batch = rad.Batch(models, precision="fp64")
    batch.run(enforce_iters=7, enforce_tol=tol)
    got = [host(m["F"]) for m in models]
    stats = batch.stats()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        batch.run(enforce_iters=7, enforce_tol=tol)
    for m, f in zip(models, start):
        m["F"].copy_(f)
    g.replay()
    torch.cuda.synchronize()
    for a, m, s, c in zip(got, models, stats, batch.stats()):
        assert np.array_equal(a, host(m["F"]))
        for key in ("iters", "converged", "closure_defect", "recip_err", "device_status"):
            assert s[key] == c[key], key


def test_bad_model_stops_alone():
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd._lib import RadError
    models = _models([300, 130, 70])
    good = [m["F"].clone() for m in models]
    models[1]["F"][100, 3] = -1.0
    bad = models[1]["F"].clone()
    batch = rad.Batch(models, precision="fp64")
    batch.run(enforce_iters=5)
    with pytest.raises(RadError) as e:
        batch.stats()
    assert e.value.code == -2
    assert torch.equal(models[1]["F"], bad)
    for k in (0, 2):
        rad.enforce_vf_(good[k], models[k]["area"], models[k]["n_rays"], tol=0.0, max_iter=5)
        assert torch.equal(models[k]["F"], good[k])
