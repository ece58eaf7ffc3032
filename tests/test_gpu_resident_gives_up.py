"""A resident enforcement whose workgroups do not wait for each other (no patience) gives up, writes
nothing, and the kernel after it does the work alone: the same bits, statistics and codes as the
streamed enforcement of a captured run."""
import numpy as np
import pytest

from tests.gpu_util import dev, need_gpu, torch

pytestmark = pytest.mark.gpu

KEYS = ("iters", "converged", "closure_defect", "recip_err", "device_status")


def _model(n, seed):
    rng = np.random.default_rng(seed + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    return F, rng.uniform(0.5, 2.0, n), rng.integers(100, 10000, n).astype(float)


def _stats(batch):
    from paper_2511_04277_amd import _lib as L
    out = (L.RadStats * batch.count)()
    L.lib().rad_batch_stats(batch._plan, batch.work.data_ptr(), out, torch.cuda.current_stream().cuda_stream)
    return [[getattr(s, k) for k in KEYS] for s in out]


@pytest.mark.parametrize("kappa", ["fracvar", "half"])
@pytest.mark.parametrize("sizes,tol,iters", [([65], 0.0, 4), ([130, 300, 64, 1], 1e-3, 12), ([700, 200], 0.0, 5),
                                             ([1500], 0.0, 3)])
@pytest.mark.parametrize("spoil", [None, "entry", "row", "area"])
def test_same_as_streamed(monkeypatch, sizes, tol, iters, kappa, spoil):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd import _lib as L
    if spoil and sizes[0] > 300:
        pytest.skip("one size is enough")
    monkeypatch.setenv("RAD_RESIDENT_PATIENCE", "0")
    models, start = [], []
    for k, n in enumerate(sizes):
        F, area, rays = _model(n, k)
        if k == 0 and spoil == "entry":
            F[n - 1, 3] = -1.0
        if k == 0 and spoil == "row":
            F[2, :] = F[:, 2] = 0.0
        if k == 0 and spoil == "area":
            area[5] = -1.0
        half = dev(np.full(n, 0.5))
        models.append({"F": dev(F), "area": dev(area), "n_rays": dev(rays), "eps": [half], "rho": [half]})
        start.append(dev(F))
    batch = rad.Batch(models, precision="fp64", kappa=kappa)
    print(f"[gives up] {sizes} {kappa} {spoil}", flush=True)
    batch.run(enforce_iters=iters, enforce_tol=tol)
    got, got_f = _stats(batch), [m["F"].clone() for m in models]
    for m, f in zip(models, start):
        m["F"].copy_(f)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        batch.run(enforce_iters=iters, enforce_tol=tol)
    g.replay()
    assert got == _stats(batch)
    good = range(1 if spoil else 0, len(models))
    for k in good:
        assert torch.equal(got_f[k], models[k]["F"])
    for k in good:
        f = start[k].clone()
        st = rad.enforce_vf_(f, models[k]["area"], models[k]["n_rays"], kappa=kappa, tol=tol, max_iter=iters)
        assert torch.equal(f, got_f[k])
        assert [st[key] for key in KEYS] == got[k]
    if spoil:
        with pytest.raises(L.RadError) as e:
            rad.enforce_vf_(start[0].clone(), models[0]["area"], models[0]["n_rays"], kappa=kappa, max_iter=iters)
        assert e.value.code == {"entry": -2, "row": -3, "area": -1}[spoil]
