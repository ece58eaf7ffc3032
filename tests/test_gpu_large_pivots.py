"""Balance matrices near the end of the range: entries below the accepted 1e300, whose row sums (the
pivots) are beyond it and finite, solve like any other."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 130, 1100])
@pytest.mark.parametrize("precision", ["fp64", "fp64_i8"])
def test_pivots_past_1e300(n, precision):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n)
    Y = rng.uniform(0.2, 1.0, (n, n + 1))
    Y *= 8.0 / Y.sum(axis=1, keepdims=True)  # rows sum to 8
    weight, Q = rng.uniform(0.5, 2.0, n), rng.uniform(0.1, 0.3, n)
    want, _, _ = rad.steady_temperature(dev(Y), dev(weight), dev(Q), sigma=1.0, t_space=1.0,
                                         precision=precision)
    # a power of two over both sides of the balance: the same temperatures, pivots of 1.3e300 to 1e301
    scale = 2.0 ** 997 * (1.0 if n > 8 else 0.125)
    got, _, _ = rad.steady_temperature(dev(Y * scale), dev(weight), dev(Q * scale), sigma=1.0, t_space=1.0,
                                         precision=precision)
    assert Y.max() * scale <= 1e300 < 8.0 * scale
    assert np.abs(host(got) / host(want) - 1).max() < 1e-12
