"""Up to 1024 faces and groups the group map is sorted in one workgroup, past that in four launches:
member order and group offsets (through the aggregated sums, bit for bit against sums in member
order) and the refusal of bad maps, around the limit."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, need_gpu, torch

pytestmark = pytest.mark.gpu


def ids(group):
    return torch.tensor(group, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("n,g", [(1, 1), (33, 32), (64, 3), (65, 64), (700, 1), (1023, 300), (1024, 1024), (1025, 300)])
def test_sums_in_member_order(n, g):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n + g)
    group = np.concatenate([np.arange(g), rng.integers(0, g, n - g)])
    rng.shuffle(group)
    X, w = rng.uniform(size=(n, n + 1)), rng.uniform(0.5, 2.0, n)
    Y, W = rad.aggregate_nodes(dev(X), dev(w), ids(group), g)
    want, ws = np.zeros((g, g + 1)), np.zeros(g)
    cols = np.zeros((n, g + 1))
    for j in range(n):  # column sums in member order, one rounding per member
        cols[:, group[j]] += X[:, j]
    cols[:, g] = X[:, n]
    for i in range(n):
        want[group[i]] += w[i] * cols[i]
        ws[group[i]] += w[i]
    want /= ws[:, None]
    assert np.array_equal(host(W), ws)
    assert np.abs(host(Y) - want).max() <= 4e-16 * n * np.abs(want).max()  # the products may be fused with the sums


@pytest.mark.parametrize("n,g", [(40, 10), (1024, 100), (1030, 100)])
def test_bad_maps_are_refused(n, g):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd._lib import RadError
    X, w = dev(np.ones((n, n + 1))), dev(np.ones(n))
    for k, bad in ((n - 1, g), (0, -1), (n // 2, None)):
        group = np.arange(n, dtype=np.int32) % g
        if bad is None:
            group[group == g - 1] = 0  # an empty group
        else:
            group[k] = bad
        with pytest.raises(RadError) as e:
            rad.aggregate_nodes(X, w, ids(group), g)
        assert e.value.code == -1
