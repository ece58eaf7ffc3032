"""Solves with at most 16 right-hand sides take their deep products in 16 x 16 tiles with K split over
a workgroup's waves; more take the wide tiles.  Steady temperatures around that width, over part of a
panel, whole panels and remainders, against the oracle.

The exchange matrix is symmetric with a fifth of every row going to space, so the balance's condition
number is below 10; n u cond = 2100 * 1.1e-16 * 10 = 2.3e-12 in T^4, a quarter of it in T, bounds the
rounding of an elimination: 1e-11 leaves a factor of ten.  The int8-emulated products round at 2^-49 of
the operands' row maxima: 1e-10.
"""
import numpy as np
import pytest

import oracle
from oracle.steady import SIGMA
from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 15, 16, 17])
@pytest.mark.parametrize("n", [120, 140, 300, 1024, 1100, 2100])
@pytest.mark.parametrize("precision", ["fp64", "fp64_i8"])
def test_widths_match_oracle(precision, n, m):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(1000 * m + n)
    S = rng.uniform(0.0, 1.0, (n, n))
    S += S.T
    w = S.sum(axis=1) / 0.8
    Y = np.concatenate([S, 0.2 * w[:, None]], axis=1) / w[:, None]
    w *= 2.0 / w.max()
    q = rng.uniform(0.0, 400.0, (n, m))
    T, _, st = rad.steady_temperature(dev(Y), dev(w), dev(q), None, t_space=3.0, sigma=SIGMA, precision=precision)
    assert st["status"] == 0
    want = oracle.steady_temperature(Y, w, q, t_space=3.0)
    assert np.abs(host(T) - want).max() < (1e-11 if precision == "fp64" else 1e-10) * want.max()
