"""The diagonal block as two 64-wide halves: a zero pivot is reported from any tile of either half,
and the L blocks of a batched step take 32 rows per workgroup past 4096 rows together, 16 below it as
the single solve does; a row's arithmetic is the same, so the REF matrices agree bitwise."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu

pytestmark = pytest.mark.gpu


def _model(n):
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    eps = rng.uniform(0.1, 0.9, n)
    return F, eps, 1.0 - eps


@pytest.mark.parametrize("k", [0, 15, 47, 63, 64, 80, 127, 128, 200])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_zero_pivot_is_reported(precision, k):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd._lib import RadError
    F, eps, rho = _model(210)
    F[k] = 0.0
    F[k, k] = 1.0  # a face that sees only itself and reflects all: row and pivot k of K are zero
    F[:k, k] = F[k + 1:, k] = 0.0
    eps[k], rho[k] = 0.0, 1.0
    with pytest.raises(RadError) as e:
        rad.gebhart_ref(dev(F), dev(eps), dev(rho), precision=precision)
    assert e.value.code == -4


@pytest.mark.parametrize("count", [8, 9])  # 512 rows below the first block of each: 4096 and 4608
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_batched_rows_per_workgroup(precision, count):
    need_gpu()
    import paper_2511_04277_amd as rad
    F, eps, rho = _model(600)
    m = {"F": dev(F), "area": dev(np.ones(600)), "n_rays": dev(np.full(600, 1e4)), "eps": [dev(eps)],
         "rho": [dev(rho)]}
    b = rad.Batch([dict(m, F=dev(F)) for _ in range(count)], precision=precision)
    b.run(ir_steps=1)
    B, _, _ = rad.gebhart_ref(dev(F), dev(eps), dev(rho), precision=precision, ir_tol=0.0, ir_max=1)
    for q in range(count):
        assert np.array_equal(host(B), host(b.B[q][0]))
