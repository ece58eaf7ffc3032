"""Aggregation and view fractions where outputs, members and rows meet the reduction kernel's other
edges: outputs per thread that do not exist (few groups, the last of 16 and 32), groups longer than the
members kept in registers, rows past half of the LDS.  All terms are positive, so a sum of at most
n + 1 of them in any order is within n eps of another order's: 10301 * 1.1e-16 = 1.2e-12 a sum, and a
quotient has two."""
import pytest

from tests.gpu_util import need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g", [(600, 17), (3000, 40), (3000, 513), (4500, 4200), (9000, 4097), (10239, 2100),
                                 (10240, 2100), (10300, 3000)])
def test_matches_index_add(n, g):
    need_gpu()
    import paper_2511_04277_amd as rad
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + g)
    X = 0.1 + torch.rand(n, n + 1, generator=gen, dtype=torch.float64, device="cuda")
    w = 0.1 + torch.rand(n, generator=gen, dtype=torch.float64, device="cuda")
    # every group a member, the rest uneven
    grp = torch.cat([torch.arange(g, device="cuda"),
                     (g * torch.rand(n - g, generator=gen, device="cuda") ** 2).long().clamp_(max=g - 1)])
    grp = grp[torch.randperm(n, generator=gen, device="cuda")]
    cols = torch.cat([grp, torch.tensor([g], device="cuda")])

    def pair_sums(rows):
        by_row = torch.zeros(g, n + 1, dtype=torch.float64, device="cuda").index_add_(0, grp, rows)
        return torch.zeros(g, g + 1, dtype=torch.float64, device="cuda").index_add_(1, cols, by_row)

    weight = torch.zeros(g, dtype=torch.float64, device="cuda").index_add_(0, grp, w)
    Y, W = rad.aggregate_nodes(X, w, grp.to(torch.int32), g)
    assert (W / weight - 1).abs().max().item() < 2.4e-12
    assert (Y / (pair_sums(X * w[:, None]) / weight[:, None]) - 1).abs().max().item() < 2.4e-12
    R = rad.view_fractions(X, grp.to(torch.int32), g)
    assert (R * pair_sums(X)[grp][:, cols] / X - 1).abs().max().item() < 2.4e-12
