"""Rows of more than 64 features that lie between two nodes to the last bit: which node they go to follows from the order in which float32 direct
differences are added up, and that order is the same in every form of the search and for any number of rows."""
import numpy as np
import pytest
import torch

from test_gpu_held_rows import som  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def tied(K, D, seed):
    """K / 2 samples, each exactly half way between two nodes of its own: whole numbers, so that every difference is exact, every product and
    sum exact in float64, and only the float32 additions round."""
    rng = np.random.default_rng(seed)
    X = rng.integers(-2 ** 14, 2 ** 14, size=(K // 2, D)).astype(np.float64)
    e = rng.integers(0, 2 ** 11, size=X.shape).astype(np.float64)
    W = np.concatenate([X + e, X - rng.permuted(e, axis=1)])
    place = rng.permutation(K)
    return X, W[np.argsort(place)], place.reshape(2, K // 2)      # sample i's nodes: place[0, i], place[1, i]


def in_order(diff, groups):
    """Float32 sums of squares, fused multiply-add by multiply-add over each of sixteen groups of features, then across the groups
    (strides 8, 4, 2, 1); one group: in the order of the features."""
    sq = diff * diff
    parts = []
    for g in groups:
        s = np.zeros(len(diff), np.float32)
        for f in g:
            s = (s.astype(np.float64) + sq[:, f]).astype(np.float32)
        parts.append(s)
    while len(parts) > 1:
        half = len(parts) // 2
        parts = [parts[i] + parts[i + half] for i in range(half)]
    return parts[0]


def choice(X, W, place, groups):
    a, b = (in_order(X - W[p], groups) for p in place)
    first = np.where((b < a) | ((b == a) & (place[1] < place[0])), 1, 0)
    return np.take_along_axis(place, first[None], 0)[0]


# held rows, rows cut beforehand, and the tile
@pytest.mark.parametrize("K,D,tile", [(400, 65, False), (1024, 200, False), (512, 256, False), (600, 257, False), (600, 330, False), (1024, 2000, False),
                                      (300, 300, True), (256, 1000, True)])
def test_sums_of_every_sixteenth_feature(som, K, D, tile):  # noqa: F811
    X, W, place = tied(K, D, K + D)
    want = choice(X, W, place, [range(p, D, 16) for p in range(16)])
    blocks = choice(X, W, place, [[f for f in range(D) if f // 4 % 16 == p] for p in range(16)])
    in_a_row = choice(X, W, place, [range(D)])
    assert (want != blocks).sum() > 20 and (want != in_a_row).sum() > 20      # the sums do tell the orders apart
    Wd = torch.from_numpy(W.astype(np.float32)).cuda()
    for copies in (1, 40):                                                    # few rows, and many of each
        Xd = torch.from_numpy(np.tile(X, (copies, 1)).astype(np.float32)).cuda()
        got = som.som_bmu(Xd, Wd)[0].cpu().numpy()
        w = np.tile(want, copies)
        # (the tile leaves up to 256 samples whose nodes are of one class to the all-nodes pass, which adds in the order of the features)
        assert ((got == w) | (tile and copies == 1) & (got == np.tile(in_a_row, copies))).all(), (got != w).sum()


@pytest.mark.parametrize("K,D", [(400, 300), (500, 600), (330, 1110)])
def test_units_do_not_go_with_the_number_of_rows(som, K, D):  # noqa: F811
    """Enough rows for the tile on maps where few rows are cut beforehand, and few of the same rows: the same units but between nodes that float32
    direct differences do not tell apart."""
    m = 131_072
    g = torch.Generator(device="cuda").manual_seed(K)
    X = torch.rand((m, D), device="cuda", generator=g)
    W = X[:K] + 0.02 * torch.randn((K, D), device="cuda", generator=g)
    W[K // 2:] = W[:K - K // 2] + 1e-5 * torch.randn((K - K // 2, D), device="cuda", generator=g)
    some = torch.randperm(m, device="cuda", generator=g)[:3000].int()
    many, few = som.som_bmu(X, W)[0][some.long()].long(), som.som_bmu(X, W, idx=some)[0].long()
    at = (many != few).nonzero()[:, 0]
    x, w = X[some[at].long()].double(), W.double()
    a, b = ((x - w[many[at]]) ** 2).sum(1), ((x - w[few[at]]) ** 2).sum(1)
    assert len(at) == 0 or ((a - b).abs() / torch.minimum(a, b)).max().item() <= (D + 4) * 2.0 ** -23


def test_units_against_float64(som):  # noqa: F811
    """Searches of all three forms, uniform and Gaussian rows, maps as given and collapsed to a fiftieth: how many units are not float64's nearest
    node, and that those are nodes which float32 direct differences do not tell apart."""
    differ = rows = 0
    for K, D in ((1024, 100), (1024, 200), (600, 300), (300, 500), (1024, 1000), (1024, 2000)):
        for uniform in (True, False):
            m = 60_000 if D <= 500 else 30_000
            g = torch.Generator(device="cuda").manual_seed(K + D + uniform)
            X = torch.rand((m, D), device="cuda", generator=g) if uniform else torch.randn((m, D), device="cuda", generator=g)
            W = X[torch.randperm(m, device="cuda", generator=g)[:K]]
            for shrink in (1.0, 0.02):
                w = (W.mean(0) + shrink * (W - W.mean(0))).contiguous()
                b = som.som_bmu(X, w)[0].long()
                for lo in range(0, m, 10_000):
                    x, v = X[lo:lo + 10_000].double(), w.double()
                    want = ((v * v).sum(1) - 2.0 * (x @ v.t())).argmin(1)
                    at = (want != b[lo:lo + 10_000]).nonzero()[:, 0]
                    best, got = ((x[at] - v[want[at]]) ** 2).sum(1), ((x[at] - v[b[lo + at]]) ** 2).sum(1)
                    assert len(at) == 0 or (got / best - 1.0).max().item() <= (D + 4) * 2.0 ** -23, (K, D, uniform, shrink)
                    differ += len(at)
                rows += m
    print(f"{differ} of {rows} units are not float64's nearest node", flush=True)
