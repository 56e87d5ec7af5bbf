"""The update's contraction in float64 on both sides of the lines between its shapes (one, two or four blocks of sixteen nodes a wavefront,
parts of the k range) and at the ends of its blocks of nodes and columns."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def som():
    from paper_2604_26555_amd import Som
    s = Som(0)
    yield s
    s.close()


@pytest.mark.parametrize("K,D", [
    (17, 64), (100, 2000), (399, 511), (400, 575), (400, 576), (401, 1023), (1023, 256), (1024, 255), (1024, 383), (1024, 384), (1025, 447),
    (1024, 448), (1100, 63), (1281, 640), (2047, 130), (2048, 62), (2049, 64),
])
@pytest.mark.parametrize("shifted", [False, True])
def test_contraction_against_float64(som, K, D, shifted):
    g = torch.Generator(device="cuda").manual_seed(K + D)
    S = torch.randn((K, D), device="cuda", dtype=torch.float64, generator=g)
    n = torch.randint(0, 50, (K,), device="cuda", generator=g)
    G = 12 * torch.rand((K, K), device="cuda", generator=g)
    W = torch.zeros((K, D), device="cuda")
    som.som_set_safeguard("shift" if shifted else "threshold")
    som.som_neighborhood_update(S, n.to(torch.uint64), G, 3.0, W)
    som.som_set_safeguard("threshold")
    h = torch.exp(-G.double() ** 2 / 18.0)
    if shifted:
        used = n > 0
        h = torch.where(used[:, None], torch.exp(-(G.double() ** 2 - torch.where(used[:, None], G.double() ** 2, torch.inf).min(0).values) / 18.0), 0.0)
    den = (h * n[:, None].double()).sum(0)[:, None]
    want, size = (h.T @ S) / den, (h.T @ S.abs()) / den
    # sums of K products of influences good to two units, in float64, and the result's own rounding to float32
    err = (W.double() - want).abs()
    assert (err <= 2.0 ** -23 * want.abs() + (K + 8) * 2.0 ** -52 * size).all(), (err - 2.0 ** -23 * want.abs()).max().item()


@pytest.mark.parametrize("K", [1, 2, 3, 4, 15, 16, 17, 31, 33, 63, 65, 129, 255, 257, 511, 513, 700, 900])
@pytest.mark.parametrize("D", [1, 48, 63, 64, 130])
def test_contraction_of_few_steps(som, K, D):
    """Wavefronts of no k-step, of part of a batch, of one, two and three."""
    test_contraction_against_float64(som, K, D, False)


@pytest.mark.parametrize("D", [20, 100])
@pytest.mark.parametrize("shifted", [False, True])
def test_influences_of_extreme_distances(som, D, shifted):
    """Distances whose influence is one, a subnormal number, zero, or of no path at all; a distance that is no number touches its own node only."""
    K = 96
    G = torch.tensor([0.0, 1e-30, 1.0, 26.0, 37.5, 38.4, 38.6, 40.0, 1e10, 3e38, torch.inf, 5.0], device="cuda").repeat(K // 12)
    G = torch.stack([G.roll(k) for k in range(K)])
    g = torch.Generator(device="cuda").manual_seed(D)
    S = torch.randn((K, D), device="cuda", dtype=torch.float64, generator=g)
    n = torch.randint(1, 9, (K,), device="cuda", generator=g)
    W = torch.zeros((K, D), device="cuda")
    som.som_set_safeguard("shift" if shifted else "threshold")
    som.som_neighborhood_update(S, n.to(torch.uint64), G, 1.0, W)
    h = torch.where(torch.isinf(G), 0.0, torch.exp(-G.double() ** 2 / 2.0))
    want, size = [(h.T @ v) / (h.T @ n.double())[:, None] for v in (S, S.abs())]
    err = (W.double() - want).abs()
    assert (err <= 2.0 ** -23 * want.abs() + (K + 8) * 2.0 ** -52 * size).all()
    G[5, 7] = torch.nan
    som.som_neighborhood_update(S, n.to(torch.uint64), G, 1.0, W)
    som.som_set_safeguard("threshold")
    assert not torch.isnan(W[:7]).any() and not torch.isnan(W[8:]).any()
    assert not torch.isnan(W[7]).any()                       # (a sum that is no number is not at least the threshold: the node stays)
