"""Enforcement with F held on chip (one tile; all tile pairs resident) against the oracle and, bitwise,
against the batch path (from 65 faces on the same tile code, from 1985 on streamed in both)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, need_gpu, padded, torch

pytestmark = pytest.mark.gpu


def _model(n, seed):
    rng = np.random.default_rng(seed + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    return F, rng.uniform(0.5, 2.0, n), rng.integers(100, 10000, n).astype(float)


@pytest.mark.parametrize("kappa", ["fracvar", "half"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 700, 1984, 1985])
def test_equals_batch_bitwise(n, kappa):
    need_gpu()
    import paper_2511_04277_amd as rad
    F, area, rays = _model(n, 5)
    f1, f2 = padded(F, n + 9), dev(F)
    st = rad.enforce_vf_(f1, dev(area), dev(rays), kappa=kappa, tol=1e-3, max_iter=12)
    b = rad.Batch([{"F": f2, "area": dev(area), "n_rays": dev(rays), "eps": [dev(np.full(n, 0.5))],
                    "rho": [dev(np.full(n, 0.5))]}], precision="fp64", kappa=kappa)
    b.run(enforce_iters=12, enforce_tol=1e-3)
    sb = b.stats()[0]
    assert np.array_equal(host(f1), host(f2))
    for key in ("iters", "converged", "closure_defect", "recip_err"):
        assert st[key] == sb[key], key


@pytest.mark.parametrize("n", [40, 300])
def test_matches_oracle_and_reports_errors(n):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd._lib import RadError
    F, area, rays = _model(n, 9)
    f = dev(F)
    rad.enforce_vf_(f, dev(area), dev(rays), max_iter=6)
    want = oracle.enforce_vf(F, area, rays, "fracvar", tol=0.0, max_iter=6)[0]
    # six steps of a few roundings on entries below one
    assert np.abs(host(f) - want).max() < 1e-14
    for spoil, code in ((lambda x: x.__setitem__((n - 1, 3), np.nan), -2),
                        (lambda x: x.__setitem__((1, n), -1.0), -2),
                        (lambda x: (x.__setitem__((2, slice(None)), 0.0), x.__setitem__((slice(None), 2), 0.0)), -3)):
        g = F.copy()
        spoil(g)
        with pytest.raises(RadError) as e:
            rad.enforce_vf_(dev(g), dev(area), dev(rays), max_iter=3)
        assert e.value.code == code
    with pytest.raises(RadError):
        rad.enforce_vf_(dev(F), dev(-area), dev(rays), max_iter=3)


def test_captured_call_replays():
    """A capture records the streamed launches (fixed iterations, no statistics)."""
    need_gpu()
    import paper_2511_04277_amd as rad
    F, area, rays = _model(200, 3)
    f0, f, a, r = dev(F), dev(F), dev(area), dev(rays)
    want = dev(F)
    rad.enforce_vf_(want, a, r, max_iter=5)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        rad.enforce_vf_(f, a, r, max_iter=5, want_stats=False)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        f.copy_(f0)
        rad.enforce_vf_(f, a, r, max_iter=5, want_stats=False)
    for _ in range(3):
        f.fill_(float("nan"))
        g.replay()
        assert torch.equal(f, want)
        torch.cuda.synchronize()
