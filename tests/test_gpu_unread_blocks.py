"""The panel inverses are triangular by 128-blocks and the blocks on the other side are neither
written nor read: what the factor buffer held before (zeros, or all bits set, i.e. NaN) leaves the
REF matrix and the gradients as they are, bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [100, 129, 300, 385, 640, 1025, 1300, 2200])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir", "fp64_i8"])
def test_old_contents_do_not_matter(precision, n):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd.api import Factors
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    eps = rng.uniform(0.1, 0.9, n)
    F, eps, rho, G = dev(F), dev(eps), dev(1.0 - eps), dev(rng.normal(size=(n, n + 1)))
    out = []
    for fill in (0, 255):
        fac = Factors(n, precision, F.device)
        fac.buf.fill_(fill)
        B, fac, _ = rad.gebhart_ref(F, eps, rho, precision=precision, ir_max=2, factors=fac)
        ge, gr, _, _ = rad.gebhart_ref_adjoint(fac, F, rho, B, G, ir_max=2)
        out.append([host(x) for x in (B, ge, gr)])
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
