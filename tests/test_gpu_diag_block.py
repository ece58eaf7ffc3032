"""Sizes around the 16-wide pivot tiles and the 128-wide diagonal block of the solve's
Gauss-Jordan inverse, against the oracle.

K is diagonally dominant with rows summing to at most 1 + max rho, so its condition
number is below (1 + rho) / (1 - rho) = 19 at rho = 0.9; n eps cond = 140 * 1.1e-16 * 19
= 3e-13 bounds the rounding of an elimination, 1e-12 leaves a factor three.  The FP32 path
stops once a correction is below 1e-12: 1e-11.
"""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 100, 112, 113, 127, 128, 129, 140])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_block_edges_match_oracle(precision, n):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(1000 + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.7)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    eps = rng.uniform(0.1, 0.9, n)
    rho = 1.0 - eps
    want = oracle.gebhart_ref(F, eps, rho)
    B, _, st = rad.gebhart_ref(dev(F), dev(eps), dev(rho), precision=precision)
    assert st["status"] == 0
    assert np.abs(host(B) - want).max() < (1e-12 if precision == "fp64" else 1e-11)
