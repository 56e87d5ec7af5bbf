"""The kernels of small calls on both sides of their limits, and the wide search, the sort and the default search at the
sizes where they can go wrong, against the oracle.

Bars as in tests/test_gpu_parity.py: units outside the 1e-5 near-tie mask identical (inside it the oracle's update follows the
GPU's unit), distances and weights within 1e-4 relative, counts exact, float64 sums within 1e-9 of max|x| n_k."""
import numpy as np
import pytest
import torch

import oracle
from synth import GaussianMixture, draw_initial_rows, draw_subset

pytestmark = pytest.mark.gpu

REL = 1e-4


@pytest.fixture(scope="module")
def som():
    from paper_2604_26555_amd import Som
    s = Som(0)
    yield s
    s.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rows(seed, m, D, n_comp=6):
    return GaussianMixture(seed, D, n_comp).rows(0, m)


def check_units(b_gpu, X, W):
    b, best, second = oracle.bmu_gram(X, W)
    mask = oracle.near_tie_mask(best, second)
    assert ((b_gpu == b) | mask).all(), f"{int(((b_gpu != b) & ~mask).sum())} wrong units outside the near-tie mask"
    return b, best, mask


def check_weights(W_gpu, W_or, den=None):
    keep = np.ones(len(W_or), dtype=bool)
    if den is not None:
        keep = ~((den > oracle.DEFAULT_EPS_H / 4) & (den < 4 * oracle.DEFAULT_EPS_H))
    err = np.abs(W_gpu.astype(np.float64) - W_or) / np.maximum(np.abs(W_or).max(axis=1, keepdims=True), 1e-30)
    assert (err[keep] <= REL).all(), f"max relative weight error {err[keep].max():.3e}"


# ---------------------------------------------------------------------------------------------------- small epochs
def epoch_against_oracle(som, X, W, G, sigma, idx=None):
    """One epoch without statistics from W; the oracle follows the GPU's units inside the near-tie mask."""
    Xd, Wd = dev(X), dev(W)
    idx_d = dev(idx.astype(np.int32)) if idx is not None else None
    Xp = X if idx is None else X[idx.astype(np.int64)]
    b_gpu = som.som_bmu(Xd, Wd, idx=idx_d)[0].cpu().numpy()
    b, _, mask = check_units(b_gpu, Xp, W)
    ref = oracle.epoch_grouped(Xp, None, W, G.astype(np.float64), sigma, b=np.where(mask, b_gpu, b))
    som.som_epoch(Xd, Wd, dev(G), sigma, idx=idx_d, want_stats=False)
    som.som_sync()
    check_weights(Wd.cpu().numpy(), ref["W"], ref["den"])
    return Wd.cpu().numpy()


def square(side):
    return oracle.rect_lattice_distances(side, side).astype(np.float32)


def line(K):
    i = np.arange(K)
    return np.abs(i[:, None] - i[None, :]).astype(np.float32)


def test_small_epochs_on_maps_that_grow_and_shrink(som):
    """The two sets of sums take turns, each cleared by the call before as far as that call's map went; a refused call
    between them changes nothing, and neither does a large epoch."""
    from paper_2604_26555_amd import SomError
    for it, (side, D, m) in enumerate([(10, 8, 3000), (7, 8, 2000), (15, 8, 3000), (15, 8, 1000), (4, 3, 50), (10, 24, 4000),
                                       (22, 8, 5000), (22, 12, 4000), (1, 5, 300), (10, 8, 1), (10, 8, 3000)]):
        X = rows(40 + it, m, D)
        W = rows(80 + it, side * side, D)
        print(f"small epoch {it}: {side} x {side} nodes, {m} x {D}", flush=True)
        epoch_against_oracle(som, X, W, square(side), 1.5)
        if it == 3:
            with pytest.raises(SomError):
                som.som_epoch(dev(X), dev(W), dev(square(side)), -1.0, want_stats=False)
            X2, W2 = rows(7, 9000, 50), rows(8, 400, 50)
            epoch_against_oracle(som, X2, W2, square(20), 2.0)


@pytest.mark.parametrize("m,K,D", [
    (375_000, 100, 8), (375_001, 100, 8),              # m K D = 3e8 and one row more
    (4000, 200, 32), (4000, 200, 33),                  # features of small_kernel
    (3000, 512, 8), (3000, 513, 8),                    # nodes of a small epoch
    (3000, 334, 32), (3000, 335, 32),                  # W and the sums in LDS
    (700, 512, 16), (700, 500, 13), (900, 300, 29),    # rows moved on in LDS (four and eight float4)
    (5000, 3, 1), (5000, 17, 2), (5000, 33, 31), (63, 64, 20), (1, 100, 8),
])
def test_small_epochs_on_both_sides_of_their_limits(som, m, K, D):
    X = rows(500 + K + D, m, D)
    W = X[draw_initial_rows(3, m, K)].copy() if K <= m else rows(501 + K, K, D)
    epoch_against_oracle(som, X, W, line(K), 1.0 + 0.02 * K)


@pytest.mark.parametrize("m,K,D", [
    (9000, 256, 7), (9000, 293, 6), (20_000, 227, 8), (20_000, 228, 8), (4097, 512, 3), (8200, 65, 31), (8200, 64, 31),   # K (D + 1) around 2048
    (40_000, 101, 8), (16_385, 16, 8), (33, 100, 8), (700, 1, 4), (700, 2, 32), (5000, 511, 15),                          # nodes left over
])
def test_small_epochs_with_one_and_eight_copies_of_the_sums(som, m, K, D):
    X = rows(600 + K + D, m, D)
    W = X[draw_initial_rows(4, m, K)].copy() if K <= m else rows(601 + K, K, D)
    epoch_against_oracle(som, X, W, line(K), 1.0 + 0.02 * K)


def test_small_epochs_with_a_row_list_and_padded_rows(som):
    X = rows(61, 6000, 10)
    idx = draw_subset(61, 0, 6000, 2500)
    W = X[draw_initial_rows(5, 6000, 81)].copy()
    epoch_against_oracle(som, X, W, square(9), 1.0, idx=idx)
    buf = np.full((6000, 13), 1e9, dtype=np.float32)
    buf[:, :10] = X
    Wa, Wb = dev(W), dev(W)
    som.som_epoch(dev(X), Wa, dev(square(9)), 1.0, want_stats=False)
    som.som_epoch(dev(buf)[:, :10], Wb, dev(square(9)), 1.0, want_stats=False)
    np.testing.assert_allclose(Wb.cpu().numpy(), Wa.cpu().numpy(), rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("eta,mu", [(0.5, 0.0), (1.0, 0.3), (0.25, 0.9)])
@pytest.mark.parametrize("safeguard", ["threshold", "shift"])
def test_small_epochs_with_momentum_and_shifted_exponents(som, eta, mu, safeguard):
    """The rule inside small_update_kernel, two epochs (the second one uses the velocity the first one wrote); sigma is small
    and two thirds of the nodes are far from every row, so denominators underflow: guarded nodes coast on their velocity, with
    shifted exponents they follow the nearest occupied nodes; one node is cut off from all others."""
    K, D, m, sigma = 100, 8, 2000, 0.08
    X = rows(71, m, D)
    W = X[draw_initial_rows(2, m, K)].copy()
    W[::3] += 500.0
    W[1::3] -= 700.0
    G = square(10).copy()
    G[37, :] = G[:, 37] = np.inf
    G[37, 37] = 0.0
    W[37] = 1e4                                                  # nobody's unit, reached by no occupied node
    V = (np.random.default_rng(1).normal(size=(K, D)) * 0.1).astype(np.float32)
    Xd, Gd, Wd, Vd = dev(X), dev(G), dev(W), dev(V)
    try:
        som.som_set_safeguard(safeguard)
        som.som_set_update_rule(eta, mu, Vd)
        for _ in range(2):
            W32, V32 = Wd.cpu().numpy().copy(), Vd.cpu().numpy().copy()
            b_gpu = som.som_bmu(Xd, Wd)[0].cpu().numpy()
            b, _, mask = check_units(b_gpu, X, W32)
            S, n = oracle.accumulate(X, None, np.where(mask, b_gpu, b), K)
            assert (n == 0).sum() > 10 and n[37] == 0                # (fewer in the second epoch: the shift fetches nodes)
            if safeguard == "threshold":
                W_or, V_or, guarded = oracle.neighborhood_update_momentum(S, n, G.astype(np.float64), sigma, W32, V32, eta, mu)
                assert guarded.any() and not guarded.all()
            else:
                target, unchanged = oracle.neighborhood_update_shifted(S, n, G.astype(np.float64), sigma, W32)
                assert unchanged.sum() == 1 and unchanged[37]
                V_or = np.where(unchanged[:, None], 0.0, eta * (target - W32)) + mu * V32
                W_or = W32 + V_or
            som.som_epoch(Xd, Wd, Gd, sigma, want_stats=False)
            som.som_sync()
            check_weights(Wd.cpu().numpy(), W_or)
            np.testing.assert_allclose(Vd.cpu().numpy(), V_or, rtol=1e-4, atol=1e-4)
    finally:
        som.som_set_update_rule(1.0, 0.0, None)
        som.som_set_safeguard("threshold")


# ---------------------------------------------------------------------------------------------------- look-ups
@pytest.mark.parametrize("m,K,D", [
    (12_288, 64, 50), (12_289, 64, 50), (4096, 512, 50), (4097, 512, 50), (2048, 1024, 64), (2049, 1024, 64),
    (1024, 700, 57), (1025, 700, 57),                  # four and eight rows a workgroup
    (3, 1, 40), (9, 511, 33), (17, 513, 44), (800, 1300, 61), (5, 2100, 64),    # W in one, two and more pieces
    (4096, 2048, 16), (4097, 2048, 16), (6144, 4096, 8), (6145, 4096, 8), (3000, 4400, 3),
    (32_767, 400, 32), (32_768, 400, 32), (65_535, 1024, 5), (65_536, 1024, 5), (1000, 512, 32), (1000, 1024, 16),
])
def test_look_ups_on_both_sides_of_their_line(som, m, K, D):
    X, W = rows(900 + K + D, m, D), rows(901 + K + D, K, D)
    X[: min(m, K, 5)] = W[: min(m, K, 5)]                       # rows that lie on a node
    if K > 20:
        W[K - 3:] = W[2:5]                                      # and nodes that exist twice: the lower index
    d2 = torch.full((m,), -1.0, device="cuda")
    qe = torch.full((2,), -1.0, dtype=torch.float64, device="cuda")
    b_gpu = som.som_bmu(dev(X), dev(W), d2=d2, qe=qe)[0].cpu().numpy()
    b, best, _ = check_units(b_gpu, X, W)
    if K > 20:
        assert (b_gpu < K - 3).all()
    same = b_gpu == b
    np.testing.assert_allclose(d2.cpu().numpy()[same], best[same], rtol=REL, atol=1e-12)
    q = qe.cpu().numpy()
    assert abs(q[0] - np.sqrt(best).sum()) <= REL * np.sqrt(best).sum() and abs(q[1] - best.sum()) <= REL * best.sum()
    assert np.array_equal(som.som_bmu(dev(X), dev(W))[0].cpu().numpy(), b_gpu)
    idx = draw_subset(7, 0, m, max(1, m // 3))
    part = som.som_bmu(dev(X), dev(W), idx=dev(idx.astype(np.int32)))[0].cpu().numpy()
    assert np.array_equal(part, b_gpu[idx.astype(np.int64)])


@pytest.mark.parametrize("m,K,bases,D", [
    (1, 64, 1, 50), (5, 63, 2, 33), (1001, 512, 3, 50), (1023, 1024, 40, 64), (1025, 1500, 7, 37), (2047, 700, 100, 52), (1000, 2100, 2, 61),
    (1001, 512, 3, 8), (4999, 100, 4, 32),
])
def test_look_ups_take_the_lowest_of_equal_nodes(som, m, K, bases, D):
    """Nodes exactly as near in the same thread, in neighbouring lanes, rows of lanes, wavefronts and pieces of W."""
    rng = np.random.default_rng(m + K + bases + D)
    base = rng.uniform(-10, 10, (bases, D)).astype(np.float32)
    W = base[rng.permutation(np.arange(K) % bases)]
    pick = rng.integers(bases, size=m)
    X = base[pick].copy()                                       # on the nodes: distance zero, whichever of them
    first = np.array([np.flatnonzero((W == b).all(1))[0] for b in base])
    X[m // 2, D // 2] = np.nan                                  # no distance is less than another: the first node
    want = first[pick]
    want[m // 2] = 0
    d2 = torch.full((m,), -1.0, device="cuda")
    b = som.som_bmu(dev(X), dev(W), d2=d2)[0].cpu().numpy()
    assert np.array_equal(b, want)
    assert (np.delete(d2.cpu().numpy(), m // 2) == 0).all()


# ---------------------------------------------------------------------------------------------------- one context, all searches
def test_searches_that_follow_each_other_on_one_context(som):
    """Narrow, wide and float32 searches, look-ups and epochs share the context's preparation and its result words: long and
    short re-decision lists after each other, in both orders, each against the oracle."""
    shapes = [(30_000, 96, 3, 50), (2000, 100, 1, 100), (300, 64, 1, 8), (20_000, 300, 1, 50), (6000, 50, 4, 130), (30_000, 96, 2, 20),
              (500, 200, 2, 64)]
    order = shapes + shapes[::-1] + [shapes[0], shapes[0], shapes[4], shapes[0]]
    data = {}
    for m, distinct, copies, D in shapes:
        X = rows(3 + D + distinct, m, D)
        W = np.concatenate([X[draw_initial_rows(5, m, distinct)]] * copies)
        data[(m, distinct, copies, D)] = (dev(X), dev(W), X, W, oracle.bmu_gram(X, W))
    for it, key in enumerate(order):
        Xd, Wd, X, W, (b, best, second) = data[key]
        som.som_set_search("float32" if it % 5 == 3 else "auto")
        som.som_profile(it % 3 == 1)                             # keeps a call off the small path
        qe = torch.empty(2, dtype=torch.float64, device="cuda")
        b_gpu = som.som_bmu(Xd, Wd, qe=qe)[0].cpu().numpy()
        som.som_profile(False)
        som.som_set_search("auto")
        assert ((b_gpu == b) | oracle.near_tie_mask(best, second)).all(), f"call {it}: {key}"
        assert (b_gpu < key[1]).all()
        assert abs(qe.cpu().numpy()[1] - best.sum()) <= REL * best.sum(), f"call {it}: {key}"


# ---------------------------------------------------------------------------------------------------- wide search
@pytest.mark.parametrize("K", [65536, 65537])
@pytest.mark.parametrize("m", [256, 257])
def test_wide_search_at_the_limits_of_its_records(som, m, K):
    """Four copies of every node inside each block of 4096, so that every sample is a tie that the joined winners leave open:
    256 of them are few enough for the all-nodes pass, 257 go through the candidate pass; above 65536 nodes the 16-bit ids
    do not reach and the all-nodes pass takes every list.  The nodes are far apart, so the answer is the lowest copy."""
    D = 66
    rng = np.random.default_rng(12)
    base = rng.normal(size=(16384, D)).astype(np.float32) * 3.0
    W = np.concatenate([np.concatenate([base[1024 * b:1024 * (b + 1)]] * 4) for b in range(16)])
    lowest = np.concatenate([4096 * b + np.arange(1024) for b in range(16)])
    if K > len(W):
        W = np.concatenate([W, np.full((1, D), 1e3, dtype=np.float32)])
    pick = rng.integers(0, 16384, size=m)
    X = (base[pick] + 0.01 * rng.normal(size=(m, D))).astype(np.float32)
    d2 = torch.empty(m, device="cuda")
    b = som.som_bmu(dev(X), dev(W), d2=d2)[0].cpu().numpy()
    assert np.array_equal(b, lowest[pick])
    want = ((X.astype(np.float64) - base[pick].astype(np.float64)) ** 2).sum(1)
    np.testing.assert_allclose(d2.cpu().numpy(), want, rtol=REL)


@pytest.mark.parametrize("m,K,D", [(500, 1700, 70), (257, 1281, 65), (255, 2560, 97), (513, 769, 128), (300, 4353, 66), (1, 700, 80),
                                   (2049, 257, 96), (100, 255, 127), (300, 40, 30_000)])
def test_wide_search_with_ragged_splits(som, m, K, D):
    """Node tiles that do not divide among the workgroups of a sample tile, last tiles of a few nodes, sample tiles of one row."""
    X, W = rows(200 + K, m, D), rows(201 + K, K, D)
    W[K - 1] = W[0]                                              # the last node of the last tile against the first
    X[0] = W[0]
    d2 = torch.empty(m, device="cuda")
    qe = torch.empty(2, dtype=torch.float64, device="cuda")
    b_gpu = som.som_bmu(dev(X), dev(W), d2=d2, qe=qe)[0].cpu().numpy()
    b, best, _ = check_units(b_gpu, X, W)
    assert b_gpu[0] == 0
    np.testing.assert_allclose(d2.cpu().numpy()[b_gpu == b], best[b_gpu == b], rtol=REL, atol=1e-12)
    assert abs(qe.cpu().numpy()[1] - best.sum()) <= REL * best.sum()


# ---------------------------------------------------------------------------------------------------- accumulation by sort
@pytest.mark.parametrize("reproducible", [False, True])
@pytest.mark.parametrize("m,K,D", [(9000, 8192, 70), (9000, 8193, 70), (5000, 16384, 66), (5000, 16385, 66), (257, 1, 200), (4097, 300, 64),
                                   (20_001, 100, 126), (2048, 77, 129), (3000, 16385, 20), (64, 8192, 50), (30_000, 40, 2001),
                                   (30_000, 2047, 70), (30_000, 2048, 70), (20_000, 2081, 66), (20_000, 2048, 600), (20_000, 2049, 600), (20_000, 33, 321), (9000, 9, 257)])
def test_accumulation_by_sort_at_its_limits(som, reproducible, m, K, D):
    """Per-node counters at the ends of their LDS, one node, one segment, many segments, sums that a call adds to."""
    X = rows(600 + K + D, m, D)
    rng = np.random.default_rng(K + D)
    b = rng.integers(0, K, size=m).astype(np.int32)
    b[rng.random(m) < 0.4] = K - 1                               # a crowded last node: many segments
    b[::97] = -1                                                 # entries outside the map are skipped
    b[5::97] = K
    inside = (b >= 0) & (b < K)
    S_or, n_or = oracle.accumulate(X[inside], None, b[inside], K)
    # (fewer than four features or more nodes than the sort's counters in a fixed order, and more slabs than the LDS kernel
    # serves: float32 partial sums, otherwise float64)
    bar = (1e-6 if K > 8192 else 1e-9) * np.abs(X).max() * np.maximum(n_or, 1)[:, None]
    som.som_set_reproducible(reproducible)
    try:
        out = []
        for _ in range(2):
            S = torch.full((K, D), 7.0, dtype=torch.float64, device="cuda")
            n = torch.full((K,), 7, dtype=torch.int64, device="cuda")
            som.som_accumulate(dev(X), dev(b), K, S, n, zero_first=True)
            assert np.array_equal(n.cpu().numpy(), n_or)
            assert (np.abs(S.cpu().numpy() - S_or) <= bar).all()
            out.append(S.cpu().numpy().copy())
        if reproducible and K <= 8192:
            assert np.array_equal(out[0], out[1])
        som.som_accumulate(dev(X), dev(b), K, S, n, zero_first=False)
        assert np.array_equal(n.cpu().numpy(), 2 * n_or)
        assert (np.abs(S.cpu().numpy() - 2 * S_or) <= 2 * bar).all()
        idx = draw_subset(9, 0, m, max(1, m // 2))
        S2, n2 = oracle.accumulate(X[idx.astype(np.int64)][inside[: len(idx)]], None, b[: len(idx)][inside[: len(idx)]], K)
        som.som_accumulate(dev(X), dev(b[: len(idx)]), K, S, n, idx=dev(idx.astype(np.int32)), zero_first=True)
        assert np.array_equal(n.cpu().numpy(), n2) and (np.abs(S.cpu().numpy() - S2) <= bar + 1e-6 * (K > 8192)).all()
    finally:
        som.som_set_reproducible(False)


@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("m,K,D", [(20_011, 300, 4), (20_011, 1025, 15), (20_011, 1100, 16), (70_001, 700, 31), (70_001, 700, 32), (999, 2300, 15),
                                   (1, 5, 7), (66, 1, 9), (257, 3, 30), (5000, 4000, 14)])
def test_accumulation_of_several_rows_together(som, listed, m, K, D):
    """Four rows of up to 15 features, two of up to 31: whole and partial batches, one and several slabs, one node for many rows."""
    gen = torch.Generator(device="cuda").manual_seed(m + K + D)
    X = torch.randn((3 * m if listed else m, D + 1), device="cuda", generator=gen)[:, :D]
    idx = torch.randperm(3 * m, device="cuda", generator=gen)[:m].int() if listed else None
    bmu = (torch.rand(m, device="cuda", generator=gen) ** 3 * K).int().clamp_(max=K - 1)
    S = torch.full((K, D), 7.0, device="cuda", dtype=torch.float64)
    n = torch.full((K,), 7, device="cuda", dtype=torch.int64)
    som.som_accumulate(X, bmu, K, S, n, idx=idx)
    rows_, b = (X if idx is None else X[idx.long()]).double().cpu().numpy(), bmu.cpu().numpy()
    want = np.zeros((K, D))
    np.add.at(want, b, rows_)
    size = np.zeros((K, D))
    np.add.at(size, b, np.abs(rows_))
    count = np.bincount(b, minlength=K)
    assert np.array_equal(n.cpu().numpy(), count)
    # n_k roundings of sums below the sum of magnitudes, on both sides
    assert (np.abs(S.cpu().numpy() - want) <= 2 * count[:, None] * 2.0 ** -53 * size).all()


@pytest.mark.parametrize("m,K,D,ldx", [(40, 16, 8, 1 << 22), (33, 300, 70, (1 << 22) + 3), (650_000, 200, 1000, 1000), (700_001, 3, 900, 900)])
def test_accumulation_by_sort_of_rows_far_apart_and_of_large_matrices(som, m, K, D, ldx):
    """Strides beyond the slab kernel's offsets; matrices beyond 2.5 GB, whose segments are shorter: float64 sums in both."""
    gen = torch.Generator(device="cuda").manual_seed(m + D)
    X = torch.empty((m - 1) * ldx + D, device="cuda").as_strided((m, D), (ldx, 1))
    X.copy_(torch.rand(m, D, generator=gen, device="cuda") - 0.5)
    b = (torch.rand(m, generator=gen, device="cuda") ** 2 * K).to(torch.int32).clamp_(max=K - 1)
    S = torch.full((K, D), 7.0, dtype=torch.float64, device="cuda")
    n = torch.full((K,), 7, dtype=torch.int64, device="cuda")
    som.som_accumulate(X, b, K, S, n, zero_first=True)
    want = torch.zeros(K, D, dtype=torch.float64, device="cuda")
    for i in range(0, m, 50_000):
        want.index_add_(0, b[i:i + 50_000].long(), X[i:i + 50_000].double())
    n_want = torch.bincount(b.long(), minlength=K)
    assert torch.equal(n, n_want)
    # both sides add up to n_k doubles: n_k units of the last place of sums below n_k / 2
    bar = n_want.double()[:, None] ** 2 * 2.0 ** -53
    assert ((S - want).abs() <= bar).all()


@pytest.mark.parametrize("m,K,bases,D", [
    (20_000, 1024, 512, 50), (20_000, 1000, 333, 25), (20_000, 1024, 256, 37),      # two, three and four nodes exactly as near: the pair list
    (3000, 1024, 256, 50), (20_000, 1024, 60, 64), (20_000, 4096, 500, 20),         # more: the candidate pass (short lists: all nodes)
    (20_000, 1024, 4, 50), (20_000, 640, 3, 64), (20_001, 130, 2, 8),               # so many that its queues overflow
    # every row on the list, so that its workgroups take two tiles, whose last stage is a partial one in the first tile's buffer
    # (K mod 256 in 33 ... 96): few candidates, and so many that the queues are served between the stages; half tiles, full ones
    (20_000, 300, 60, 50), (20_000, 576, 96, 37), (20_001, 340, 68, 20), (20_000, 300, 25, 50), (20_000, 576, 48, 37), (150_000, 289, 29, 12),
])
def test_bmu_exact_ties_over_many_nodes(som, m, K, bases, D):
    """Every node is one of `bases` rows far apart, so each sample has K / bases winners that are exactly as near: the lowest index,
    whichever of the re-decisions finds it and wherever the rows lie in the stages."""
    rng = np.random.default_rng(m + K + bases + D)
    base = rng.uniform(-10, 10, (bases, D)).astype(np.float32)
    W = base[rng.permutation(np.arange(K) % bases)]
    X = (base[rng.integers(bases, size=m)] + rng.normal(size=(m, D)) * 0.05).astype(np.float32)
    first = np.array([np.flatnonzero((W == b).all(1))[0] for b in base])
    near = np.concatenate([((x[:, None, :].astype(np.float64) - base[None].astype(np.float64)) ** 2).sum(2).argmin(1)
                           for x in np.array_split(X, max(1, m * bases * D // 10_000_000))])
    b, _, _ = som.som_bmu(dev(X), dev(W))
    assert np.array_equal(b.cpu().numpy(), first[near])


@pytest.mark.parametrize("m,K,D,run", [(20_000, 300, 50, 32), (20_000, 320, 64, 32), (20_000, 577, 50, 32), (150_000, 289, 12, 64)])
def test_bmu_exact_ties_uneven_among_wavefronts(som, m, K, D, run):
    """One wavefront of four has samples of 40 equally near nodes, the others of five: they are far apart when a workgroup goes on to its
    next tile (every row is listed; last stages as above)."""
    rng = np.random.default_rng(m + K + D)
    heavy = 2
    base = rng.uniform(-10, 10, (heavy + -(-(K - 40 * heavy) // 5), D)).astype(np.float32)
    of = np.concatenate([np.repeat(np.arange(heavy), 40), heavy + np.arange(K - 40 * heavy) // 5])
    W = base[of[rng.permutation(K)]]
    many = np.arange(m) // run % 4 == 0
    near = np.where(many, rng.integers(heavy, size=m), rng.integers(heavy, len(base), size=m))
    X = (base[near] + rng.normal(size=(m, D)) * 0.05).astype(np.float32)
    first = np.array([np.flatnonzero((W == b).all(1))[0] for b in base])
    b, _, _ = som.som_bmu(dev(X), dev(W))
    assert np.array_equal(b.cpu().numpy(), first[near])


@pytest.mark.parametrize("m,K,D", [(20_000, 512, 17), (20_000, 512, 50), (20_000, 512, 64), (20_000, 512, 100)])
def test_bmu_where_squares_of_the_parts_underflow(som, m, K, D):
    """Rows of about 10^-17: what the first bf16 part leaves over has squares around the smallest normal number, below which the
    hardware's root returns zero; every node has another one close by, so that the bounds formed from those squares decide who is listed."""
    rng = np.random.default_rng(D)
    base = rng.uniform(-10, 10, (K // 2, D))
    W = (np.concatenate([base, base + rng.normal(size=base.shape) * 0.02]) * 2.0 ** -58).astype(np.float32)
    X = ((base[rng.integers(K // 2, size=m)] + rng.normal(size=(m, D)) * 0.05) * 2.0 ** -58).astype(np.float32)
    b, _, _ = som.som_bmu(dev(X), dev(W))
    check_units(b.cpu().numpy(), X, W)


@pytest.mark.parametrize("shape,K", [("chain", 2), ("chain", 3), ("chain", 65), ("chain", 1500), ("star", 4), ("star", 70), ("star", 300),
                                     ("comb", 66), ("comb", 513), ("random", 1), ("random", 1025), ("random", 2500),
                                     # a wavefront's and a workgroup's share of the tour, and one edge more
                                     ("random", 33), ("random", 34), ("star", 513), ("random", 513), ("chain", 514), ("hubs", 1026),
                                     ("random", 2048), ("chain", 2049), ("random", 2049), ("hubs", 2048), ("hubs", 2049)])
def test_spanning_tree_hops_of_every_shape(som, shape, K):
    """The order of a spanning tree's nodes: long branches, nodes with very many branches, both mixed, and sizes around a wavefront."""
    rng = np.random.default_rng(K)
    if shape == "chain":                                    # along a line, in a mixed order
        W = (np.sort(rng.uniform(0, 10 * K, K))[rng.permutation(K)])[:, None]
    elif shape == "star":                                   # leaves 10 to 11 from the hub, at least 14 from each other
        W = np.zeros((K, K))
        W[np.arange(1, K), np.arange(1, K)] = 10 + np.arange(1, K) / K
        W = W[rng.permutation(K)]
    elif shape == "comb":                                   # a spine with teeth of four nodes
        i = np.arange(K)
        W = np.stack([(i // 5) * 3.0 + 0.001 * (i // 5) ** 1.1, (i % 5) * (1.0 + 0.0005 * i)], 1)
    elif shape == "hubs":                                   # eight far apart, every other node around one of them
        W = 1000.0 * np.eye(8, 64)[np.arange(K) % 8] + rng.normal(size=(K, 64)) * (np.arange(K) >= 8)[:, None]
    else:
        W = rng.normal(size=(K, 6))
    W = W.astype(np.float32)
    T = som.som_topology(dev(W), "mst").cpu().numpy()
    assert np.array_equal(T, oracle.graph_distances("mst", W).astype(np.float32))


@pytest.mark.parametrize("shape", ["random", "chain"])
def test_spanning_tree_where_a_node_holds_no_number(som, shape):
    """More nodes than Boruvka's rounds take, one of them NaN: no distance of its own is below another, so it stays apart, and
    the edges that are left are no tree of all nodes.  Their hop counts are searched breadth first."""
    from scipy.sparse import csr_matrix
    from scipy.sparse.csgraph import shortest_path
    K, bad = 4100, 77
    W = rows(19, K, 3, 4) if shape == "random" else np.random.default_rng(19).permutation(K).astype(np.float32)[:, None] * np.ones(3, np.float32)
    keep = np.delete(np.arange(K), bad)
    e = keep[oracle.mst_edges(W[keep])]
    W[bad, 1] = np.nan
    T = som.som_topology(dev(W), "mst").cpu().numpy()
    adj = np.zeros((K, K), dtype=bool)
    adj[e[:, 0], e[:, 1]] = adj[e[:, 1], e[:, 0]] = True
    assert np.array_equal(T == 1, adj)
    assert np.isinf(T[bad, keep]).all() and np.isinf(T[keep, bad]).all() and (T.diagonal() == 0).all()
    src = [0, bad, 1234, K - 1]
    hops = shortest_path(csr_matrix(adj.astype(np.int8)), unweighted=True, indices=src)
    assert np.array_equal(T[src], hops.astype(np.float32))


@pytest.mark.parametrize("K", [9045, 9046, 9102, 9103])
def test_spanning_tree_hops_at_the_limit_of_lds(som, K):
    """A chain of the most nodes whose tour fits 160 KB, and of more, which go breadth first."""
    place = torch.randperm(K, generator=torch.Generator().manual_seed(K)).cuda()
    T = som.som_topology(place.float()[:, None].contiguous(), "mst")
    for lo in range(0, K, 1024):
        assert torch.equal(T[lo:lo + 1024], (place[lo:lo + 1024, None] - place[None]).abs().float())


@pytest.mark.parametrize("K", [6124, 6125, 6500, 6653, 9103, 12000])
def test_neighbourhood_graph_hops_on_both_sides_of_the_lists_limit(som, K):
    """Nodes along a line: breadth first with the adjacency lists in LDS, and in memory where they would crowd out the sources."""
    place = torch.randperm(K, generator=torch.Generator().manual_seed(K)).cuda()
    T = som.som_topology(place.float()[:, None].contiguous(), "rng")
    for lo in range(0, K, 1024):
        assert torch.equal(T[lo:lo + 1024], (place[lo:lo + 1024, None] - place[None]).abs().float())


def test_neighbourhood_graphs_of_many_nodes_cost_no_more_per_pair(som):
    """Graphs of 9000 nodes against 6000 (2.25 times the pairs): nine times as long a call when the lists left room for one source to a compute
    unit, three times without them."""
    times = []
    for K in (6000, 9000):
        W = torch.randn((K, 8), device="cuda", generator=torch.Generator(device="cuda").manual_seed(K))
        G = torch.empty((K, K), device="cuda")
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            som.som_topology(W, "rng", G=G)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"6000 nodes {times[0]:.2f} ms, 9000 {times[1]:.2f}", flush=True)
    assert times[1] < 5 * times[0], times


@pytest.mark.parametrize("K", [33, 128, 129, 300, 384, 385, 513])
@pytest.mark.parametrize("D", [53, 60, 64])
def test_four_blocks_of_features_on_both_sides_of_the_short_maps_limit(som, D, K):
    """Scores folded two at a time (up to 384 nodes) and four at a time, through the search, its pair list and its candidate pass (nodes in
    pairs a ten-thousandth apart, so that samples are listed)."""
    m = 500_000_000 // (K * D)
    X = rows(900 + K + D, m, D)
    W = rows(901 + K + D, K, D)
    W[K // 2:2 * (K // 2)] = W[:K // 2] + 1e-4 * np.random.default_rng(K).normal(size=(K // 2, D)).astype(np.float32)
    check_units(som.som_bmu(dev(X), dev(W))[0].cpu().numpy(), X, W)
