"""The search of 21 to 64 features by half-precision and fp6 parts, which large calls take, against float64 and against the same rows
presented in pieces small enough for the two bf16 parts.

Either way a sample whose best two scores lie inside the rounding bound is decided by direct float32 differences, features in order, so the
units are the same, bit for bit; a bound that is too small shows as a difference.  (Samples some hundred times as far out as the nodes lie from one
another are told apart by the scores better than by those differences: there the wider of two bounds may show, the one exception that
include/som.h names.)  Against float64, a float32 sum of
D squared differences is off by at most (D + 2) * 2^-24 of itself, so a unit may only miss the nearest node where the two distances are closer
than twice that.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def som():
    from paper_2604_26555_amd import Som
    s = Som(0)
    yield s
    s.close()


def rows_for(K, D):
    """Rows that take the call to these parts, and a piece that does not (the rule of half_parts_pay: rows times MFMAs saved a row)."""
    left = D % 16
    two = 3 * (D // 16) + 1 if 1 <= left <= 4 else 3 * ((D + 15) // 16)
    fewer = (K + 31) // 32 * (two - (D + 31) // 32 - ((D + 3) // 4 // 4 + 1))
    assert fewer >= 40, "no such map"
    return 40_000_000 // fewer + 7, 40_000_000 // fewer // 3


def check(som, X, W, idx=None, same=True):
    K, D = W.shape
    m = X.shape[0] if idx is None else idx.numel()
    whole, _, _ = som.som_bmu(X, W, idx=idx)
    whole = whole.clone()
    _, piece = rows_for(K, D)
    parts = []
    for lo in range(0, m, piece):
        hi = min(m, lo + piece)
        b, _, _ = som.som_bmu(X[lo:hi] if idx is None else X, W, idx=None if idx is None else idx[lo:hi])
        parts.append(b.clone())
    differ = whole != torch.cat(parts)
    if not same:
        differ &= (torch.linalg.norm(X - W.mean(0), dim=1) < 100 * torch.linalg.norm(W - W.mean(0), dim=1).max())
    assert not differ.any(), int(differ.sum())
    return whole


def against_float64(X, W, units):
    w, D = W.double(), W.shape[1]
    c = w.mean(0)
    worst = 0.0
    for lo in range(0, X.shape[0], 16384):
        x = X[lo:lo + 16384].double()
        d = ((x - c) ** 2).sum(1)[:, None] - 2 * (x - c) @ (w - c).t() + ((w - c) ** 2).sum(1)
        own = ((x - w[units[lo:lo + 16384].long()]) ** 2).sum(1)
        least = d.min(1).values
        worst = max(worst, float(((own - least) / own.clamp_min(1e-300)).max()))
    assert worst <= 2 * (D + 2) * 2.0 ** -24, worst


@pytest.mark.parametrize("D,K", [(21, 1024), (24, 1025), (25, 449), (28, 1151), (29, 2500), (32, 700), (33, 1300), (36, 1024), (37, 437), (44, 1100),
                                 (45, 1030), (48, 1089), (49, 640), (50, 4096), (52, 321), (53, 1024), (60, 300), (61, 1024), (64, 999)])
def test_units_of_every_form(som, D, K):
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(D * 7919 + K)
    W = torch.randn((K, D), device=DEV, generator=g) * 3 + 11
    X = W[torch.randint(K, (m,), device=DEV, generator=g)] * 0.7 + 3 + torch.randn((m, D), device=DEV, generator=g)
    against_float64(X, W, check(som, X, W))


@pytest.mark.parametrize("regime", ["collapsed", "pairs", "far samples", "far node", "tiny", "huge", "near the middle", "no numbers"])
def test_units_of_uneven_values(som, regime):
    K, D = 1100, 50
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(5)
    randn = lambda *s: torch.randn(s, device=DEV, generator=g)
    W, X = randn(K, D), 2 * randn(m, D)
    numbers = True
    if regime == "collapsed":                              # samples a thousand times as far out as the nodes lie from one another
        W = 5 + 1e-3 * W
    elif regime == "pairs":                                # every node has a neighbour a few units of the last place of a score away
        W[K // 2:] = W[:K // 2] + 1e-5 * randn(K // 2, D)
    elif regime == "far samples":
        X[::97] *= 1e5
    elif regime == "far node":                             # past what half precision holds at the other nodes' scale
        W[17] *= 1e4
        X[::1009] = W[17] + randn(X[::1009].shape[0], D)
    elif regime == "tiny":
        W, X = W * 1e-17, X * 1e-17
    elif regime == "huge":
        W, X = W * 1e15, X * 1e15
    elif regime == "near the middle":
        X *= 1e-4
    else:
        X[::101, 3] = float("nan")
        X[::103, 49] = float("inf")
        X[::107] = 3e38
        numbers = False
    units = check(som, X, W, same=regime not in ("collapsed", "far samples"))
    assert int(units.min()) >= 0 and int(units.max()) < K
    if numbers and regime != "tiny":                       # (squares of 10^-17 are all but subnormal)
        against_float64(X, W, units)


@pytest.mark.parametrize("out", [30.0, 300.0, 2000.0, 2e4, 1e6, 1e12, float("inf")])
def test_units_with_outlying_nodes(som, out):
    """Nodes inside and outside of what half precision holds at the scale of the others (some 5800 times as far out), samples near them and
    halfway to them among the rest."""
    K, D = 1100, 50
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(8)
    randn = lambda *s: torch.randn(s, device=DEV, generator=g)
    W, X = randn(K, D), 2 * randn(m, D)
    W[17] *= out
    W[900] *= 3 * out
    far = W.clone()
    if out == float("inf"):                                # a node that no sample is near, its distances infinite
        W[17] = W[900] = out
        far[17] = far[900] = 1e18
    else:
        for step, node in ((1009, 17), (1013, 900)):
            X[::step] = W[node] + randn(X[::step].shape[0], D)
            X[1::step] = W[node] * torch.rand((X[1::step].shape[0], 1), device=DEV, generator=g)
    units, w = check(som, X, W).long(), far.double()
    for lo in range(0, m, 16384):                          # (the four nearest by products, by differences among those: products of far rows round)
        x = X[lo:lo + 16384].double()
        four = ((w ** 2).sum(1) - 2 * x @ w.t()).topk(4, largest=False).indices
        least = ((x[:, None] - w[four]) ** 2).sum(2).min(1).values
        own = ((x - w[units[lo:lo + 16384]]) ** 2).sum(1)
        assert ((own - least) / own.clamp_min(1e-300)).max() <= 2 * (D + 2) * 2.0 ** -24


def test_an_outlying_node_costs_no_call(som):
    """One node far out leaves the others' samples to the matrix pipe (they took seventeen times as long when its norm decided for all)."""
    K, D, m = 1024, 50, 500_000
    g = torch.Generator(device=DEV).manual_seed(10)
    base, X = torch.randn((K, D), device=DEV, generator=g), torch.randn((m, D), device=DEV, generator=g)
    b = torch.empty(m, dtype=torch.int32, device=DEV)

    def best_of(W):
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                som.som_bmu(X, W, bmu=b)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    plain = best_of(base)
    for out in (50.0, 1000.0, 1e5):
        W = base.clone()
        W[17] *= out
        t = best_of(W)
        print(f"node times {out:g}: {t / 4 * 1e3:.0f} us, {plain / 4 * 1e3:.0f} without", flush=True)
        assert t < 3 * plain, (out, t, plain)


def test_streamed_epochs_take_the_parts_of_resident_ones(som):
    """Samples a thousand times as far out as the nodes lie from one another, where the two forms' units differ: one node of some 250 samples
    that gets one more or less moves by far more than the last places of its weights."""
    K, D = 1089, 50
    m, piece = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(12)
    W, X = 5 + 1e-3 * torch.randn((K, D), device=DEV, generator=g), 2 * torch.randn((m, D), device=DEV, generator=g)
    at = torch.arange(K, device=DEV, dtype=torch.float32)
    G = (at[:, None] - at[None, :]).abs()
    Wr, Ws = W.clone(), W.clone()
    som.som_epoch(X, Wr, G, 0.3)
    som.som_epoch_host(X.cpu().numpy(), Ws, G, 0.3, chunk_rows=piece)
    torch.cuda.synchronize()
    assert (Wr - Ws).abs().max() <= 2.0 ** -22 * Wr.abs().max()


def test_listed_rows_of_a_wider_matrix(som):
    K, D = 1024, 37
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(9)
    wide = torch.randn((m + 1000, D + 6), device=DEV, generator=g)
    X = wide[:, 3:3 + D]
    W = torch.randn((K, D), device=DEV, generator=g)
    idx = torch.randperm(m + 1000, device=DEV, generator=g)[:m].int().contiguous()
    units = check(som, X, W, idx=idx)
    against_float64(X[idx.long()], W, units)


def centre_nodes(K):
    """The sixty-four nodes whose mean the search of up to 64 features takes off samples and weights."""
    nodes = []
    for t in range(64):
        h = t * 0x9E3779B1 & 0xFFFFFFFF
        h ^= h >> 15
        h = h * 0x85EBCA77 & 0xFFFFFFFF
        h ^= h >> 13
        nodes.append(t * K // 64 + (h * (K // 64) >> 32))
    return nodes


@pytest.mark.parametrize("size", [1e-17, 1e-18, 1e-19, 3e-20, 1e-20, 1e-21, 1e-22])
def test_units_of_tiny_values(som, size):
    """Rows whose squares are subnormal or nearly so: a unit's squared distance lies above the least one by what a float32 sum of D squares
    of that size can lose: (D + 2) * 2^-24 of itself and half of 2^-149 for each of D squares and D additions, for either of the two."""
    K, D = 1100, 50
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(6)
    W, X = torch.randn((K, D), device=DEV, generator=g) * size, torch.randn((m, D), device=DEV, generator=g) * (2 * size)
    units, _, _ = som.som_bmu(X, W)
    w = W.double()
    over = 0.0
    for lo in range(0, m, 65536):
        x = X[lo:lo + 65536].double()
        d = ((x / size) ** 2).sum(1)[:, None] - 2 * (x / size) @ (w / size).t() + ((w / size) ** 2).sum(1)
        least = ((x - w[d.argmin(1)]) ** 2).sum(1)
        own = ((x - w[units[lo:lo + 65536].long()]) ** 2).sum(1)
        over = max(over, float(((own - least) / (2 * ((D + 2) * 2.0 ** -24 * own + D * 2.0 ** -149))).max()))
    assert over <= 1.0, over


@pytest.mark.parametrize("K,D", [(1100, 50), (1024, 25), (4096, 33)])
def test_scores_of_zero(som, K, D):
    """A sample halfway between the centre and its node scores x . w - |w|^2 / 2 = 0 there, and all are small whole numbers of 1/128, so
    exactly zero: a number whose low bits, which carry the node's place, do not survive any scaling."""
    m, _ = rows_for(K, D)
    g = torch.Generator(device=DEV).manual_seed(K + D)
    W = torch.randint(-1, 2, (K, D), device=DEV, generator=g).float()
    c = W[torch.tensor(centre_nodes(K), device=DEV)].mean(0)
    want = torch.arange(m, device=DEV) % K
    X = (c + W[want]) / 2
    units, _, _ = som.som_bmu(X, W)
    differ = units.long() != want
    assert not differ.any(), int(differ.sum())
