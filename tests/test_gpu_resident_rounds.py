"""The resident enforcement exchanges sums, scales and states through buffers that are used in
turn (two and four iterations): every iteration count over two rounds of them, and a long run,
bitwise against the batch path, whose group launch has an exchange of the same kind."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,iters", [(130, k) for k in range(1, 10)] + [(65, 333), (700, 64), (1984, 10)])
def test_iteration_counts(n, iters):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    area, rays = dev(rng.uniform(0.5, 2.0, n)), dev(rng.integers(100, 10000, n).astype(float))
    f1, f2 = dev(F), dev(F)
    st = rad.enforce_vf_(f1, area, rays, tol=0.0, max_iter=iters)
    b = rad.Batch([{"F": f2, "area": area, "n_rays": rays, "eps": [dev(np.full(n, 0.5))],
                    "rho": [dev(np.full(n, 0.5))]}], precision="fp64")
    b.run(enforce_iters=iters)
    sb = b.stats()[0]
    assert np.array_equal(host(f1), host(f2))
    for key in ("iters", "converged", "closure_defect", "recip_err"):
        assert st[key] == sb[key], key
    assert st["iters"] == iters
