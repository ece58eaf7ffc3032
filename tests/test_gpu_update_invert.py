"""The update by one diagonal block and the inversion of the next share a launch where the side
stream is free; the batch path has a launch of each.  The REF matrices agree bitwise for one to nine
blocks, the first panels of larger models, and repeated solves in one workspace."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [129, 257, 500, 768, 897, 1153, 2049, 3100])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_equals_batch_bitwise(precision, n):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    eps = rng.uniform(0.1, 0.9, n)
    F, eps, rho = dev(F), dev(eps), dev(1.0 - eps)
    m = {"F": F, "area": dev(np.ones(n)), "n_rays": dev(np.full(n, 1e4)), "eps": [eps], "rho": [rho]}
    b = rad.Batch([m], precision=precision)
    b.run(ir_steps=1)
    want = host(b.B[0][0])
    for _ in range(3):
        B, _, _ = rad.gebhart_ref(F, eps, rho, precision=precision, ir_tol=0.0, ir_max=1)
        assert np.array_equal(host(B), want)
