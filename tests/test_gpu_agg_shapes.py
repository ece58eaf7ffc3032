"""Aggregation, view fractions and node emissivity at the edges of the reduction kernel: row lengths
around its 512-entry pieces, every number of outputs per thread, group sizes around the members it
keeps in registers.  All terms are positive, so a sum of at most n + 1 of them in any order is within
n eps of the oracle's: 9001 * 1.1e-16 = 1e-12 per sum, and a quotient has two."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, need_gpu, padded, torch

pytestmark = pytest.mark.gpu


def _groups(rng, n, g):
    """Every group at least one member, the rest uneven."""
    grp = np.concatenate([np.arange(g), (g * rng.beta(0.6, 2.0, n - g)).astype(int)]).astype(np.int32)
    rng.shuffle(grp)
    return grp


@pytest.mark.parametrize("n,g", [(1, 1), (63, 1), (511, 511), (512, 40), (513, 513), (1023, 600), (1025, 1025),
                                 (2100, 2049), (4097, 4096), (8193, 17), (8700, 8200)])
def test_matches_oracle(n, g):
    need_gpu()
    import paper_2511_04277_amd as rad
    rng = np.random.default_rng(n * 7 + g)
    X = rng.uniform(0.1, 1.0, (n, n + 1))
    eps, area = rng.uniform(0.1, 0.9, n), rng.uniform(0.5, 2.0, n)
    grp = _groups(rng, n, g)
    x, gd = padded(X, n + 6), dev(grp, torch.int32)
    Y, W = rad.aggregate_nodes(x, dev(eps * area), gd, g)
    want, wantw = oracle.aggregate_nodes(X, eps * area, grp, g)[:2]
    assert np.abs(host(Y) / want - 1).max() < 2e-12 and np.abs(host(W) / wantw - 1).max() < 2e-12
    R = host(rad.view_fractions(x, gd, g))
    assert np.abs(R / oracle.view_fractions(X, grp, g) - 1).max() < 2e-12
    E = host(rad.node_emissivity(x, dev(eps), dev(area), gd, g))
    assert np.abs(E / oracle.node_emissivity(X, eps, area, grp, g) - 1).max() < 4e-12
