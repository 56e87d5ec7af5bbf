"""The error band of the search for rows of up to 64 features, whose width goes with the sample's distance from its winner and not with its
distance from the map's middle: choices against float64 where the two are far apart, and for candidates in pairs and crowds."""
import pytest
import torch

from test_gpu_held_rows import check, som  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 5, 15, 16, 17, 20, 21, 32, 33, 37, 48, 50, 52, 53, 64])
def test_close_nodes_far_from_the_middle(som, D):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(D)
    r = lambda *s: torch.randn(s, device="cuda", generator=g)
    for spread, gap, noise in ((30.0, 1e-1, 0.3), (30.0, 1e-2, 0.03), (300.0, 1e-2, 1e-2), (30.0, 1e-3, 1e-3), (30.0, 1e-4, 0.3), (1.0, 1e-5, 1e-5), (3.0, 1e-2, 30.0)):
        base = spread * r(60, D)
        crowd = base[:2].repeat_interleave(40, 0)
        W = torch.cat([base, base + gap * r(60, D), base[:40] + gap * r(40, D), crowd + gap * r(80, D)]).contiguous()
        X = W[torch.randint(240, (20_000,), device="cuda", generator=g)] + noise * r(20_000, D)
        check(som, X, W)


@pytest.mark.parametrize("D", [8, 50, 64])
def test_one_node_far_from_the_others(som, D):  # noqa: F811
    """The largest norms are those of a node that no sample is near to; samples on it, beside it and half way."""
    g = torch.Generator(device="cuda").manual_seed(D)
    W = torch.randn((130, D), device="cuda", generator=g)
    W[77] *= 1e4
    X = W[torch.randint(130, (20_000,), device="cuda", generator=g)] + 0.1 * torch.randn((20_000, D), device="cuda", generator=g)
    X[::5] = 0.5 * W[77] + torch.randn((4000, D), device="cuda", generator=g)
    check(som, X, W.contiguous())


@pytest.mark.parametrize("K", [1023, 1024, 1100, 2900])
@pytest.mark.parametrize("D", [5, 16, 17, 32, 50, 64])
def test_two_to_nine_close_nodes(som, D, K):  # noqa: F811
    """Groups of two to nine nodes close together, so that samples have any number of candidates among their class winners: on both sides of
    the size from which eight of them are kept, in short lists, rows in order and by a list."""
    g = torch.Generator(device="cuda").manual_seed(D + K)
    r = lambda *s: torch.randn(s, device="cuda", generator=g)
    size = 2 + torch.arange(K, device="cuda") % 8
    group = torch.repeat_interleave(torch.arange(K, device="cuda"), size)[:K]
    W = (5.0 * r(K, D))[group] + 1e-5 * r(K, D)
    W = W[torch.randperm(K, device="cuda", generator=g)].contiguous()
    for m in (70, 9000):
        X = W[torch.randint(K, (m,), device="cuda", generator=g)] + 0.1 * r(m, D)
        check(som, X, W)
        check(som, X, W, torch.randint(m, (m,), device="cuda", generator=g).int())


@pytest.mark.parametrize("candidates", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("K,D", [(1024, 16), (1024, 32), (1152, 50), (512, 50)])
def test_pair_lists_of_several_rounds(som, K, D, candidates):  # noqa: F811
    """Every row is on the pair list, three rounds of it (512 workgroups of eight wavefronts take 65,536 entries a round): the first `candidates` of every eight nodes in a row, which fall into eight classes, are close together.  Entries
    of more than two wait among those of the rounds after theirs.  (On 512 nodes those of more than four go to the candidate pass.)"""
    m = 140_000
    g = torch.Generator(device="cuda").manual_seed(K + D + candidates)
    r = lambda *s: torch.randn(s, device="cuda", generator=g)
    base = 5.0 * r(K, D).view(K // 8, 8, D)
    base[:, :candidates] = base[:, :1] + 1e-5 * r(K // 8, candidates, D)
    W = base.view(K, D).contiguous()
    eight = torch.randint(K // 8, (m,), device="cuda", generator=g)
    X = base[eight, 0] + 0.1 * r(m, D)
    for idx in (None, torch.randperm(m, device="cuda", generator=g)[:m - 5].int()):
        b = som.som_bmu(X, W, idx=idx)[0].long()
        rows = slice(None) if idx is None else idx.long()
        x, near = X[rows].double(), base[eight[rows], :candidates].double()
        nearest = ((x[:, None, :] - near) ** 2).sum(2).min(1).values
        got = ((x - W[b].double()) ** 2).sum(1)
        assert (got / nearest - 1.0).max().item() <= (D + 4) * 2.0 ** -23
