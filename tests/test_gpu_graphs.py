"""Calls recorded into a HIP graph and replayed: every replay must give what the same call gives eagerly, whatever ran on the
context between the replays.  (The workspaces are grown by an eager call first: nothing can be allocated under capture.)"""
import numpy as np
import pytest
import torch

import oracle
from synth import GaussianMixture, draw_initial_rows

pytestmark = pytest.mark.gpu

REPLAYS = 4


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Captured:
    """A context on a stream of its own; record() captures fn once, replays() yields after every replay."""

    def __init__(self):
        from paper_2604_26555_amd import Som
        self.stream = torch.cuda.Stream()
        self.som = Som(0, stream=self.stream)

    def eager(self, fn):
        with torch.cuda.stream(self.stream):
            fn()
        self.stream.synchronize()

    def record(self, fn):
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph, stream=self.stream):
            fn()
        torch.cuda.synchronize()

    def replays(self, between):
        for r in range(REPLAYS):
            with torch.cuda.stream(self.stream):
                self.graph.replay()
            self.stream.synchronize()
            yield r
            self.eager(between)

    def close(self):
        self.graph = None
        self.som.close()


@pytest.fixture
def cap():
    c = Captured()
    yield c
    c.close()


# (m, distinct nodes, copies of each, D): lists of every sample (candidate pass, pair list), none, wide rows, few rows
@pytest.mark.parametrize("search", ["auto", "float32"])
@pytest.mark.parametrize("m,distinct,copies,D", [(30_000, 96, 3, 50), (30_000, 200, 2, 20), (20_000, 300, 1, 33), (6_000, 96, 2, 130),
                                                 (500, 64, 2, 50), (300, 100, 1, 8)])
def test_replayed_searches(cap, search, m, distinct, copies, D):
    X = GaussianMixture(5 + D, D, 5).rows(0, m)
    W = np.concatenate([X[draw_initial_rows(3, m, distinct)]] * copies)
    Xd, Wd = dev(X), dev(W)
    X2, W2 = dev(X[: m // 2] * 0.5), dev(W[: len(W) // 2 + 1] * 0.25)
    bmu = torch.empty(m, dtype=torch.int32, device="cuda")
    d2 = torch.empty(m, device="cuda")
    qe = torch.empty(2, dtype=torch.float64, device="cuda")
    other = torch.empty(m // 2, dtype=torch.int32, device="cuda")
    cap.som.som_set_search(search)
    call = lambda: cap.som.som_bmu(Xd, Wd, bmu=bmu, d2=d2, qe=qe)
    print(f"replayed search: {search} m={m} K={len(W)} D={D}", flush=True)
    cap.eager(call)
    want = bmu.cpu().numpy().copy(), d2.cpu().numpy().copy(), qe.cpu().numpy().copy()
    b, best, second = oracle.bmu(X, W)
    assert ((want[0] == b) | oracle.near_tie_mask(best, second)).all()
    cap.record(call)
    for r in cap.replays(lambda: cap.som.som_bmu(X2, W2, bmu=other)):
        assert np.array_equal(bmu.cpu().numpy(), want[0]), f"replay {r}"
        assert np.array_equal(d2.cpu().numpy(), want[1]), f"replay {r}"
        np.testing.assert_allclose(qe.cpu().numpy(), want[2], rtol=1e-12)       # (the order of the float64 sums varies)
        for t in (bmu, d2, qe):
            t.fill_(-1)
        torch.cuda.synchronize()
    cap.eager(call)
    assert np.array_equal(bmu.cpu().numpy(), want[0])


# rows cut beforehand (every sample listed; none), rows held in registers on a map of several stages, five and eight candidates a sample
@pytest.mark.parametrize("m,distinct,copies,D", [(6_000, 180, 2, 300), (4_000, 400, 1, 513), (6_000, 300, 2, 200),
                                                 (20_000, 256, 5, 50), (20_000, 160, 8, 50)])
def test_replayed_searches_of_wide_rows_and_many_candidates(cap, m, distinct, copies, D):
    test_replayed_searches(cap, "auto", m, distinct, copies, D)


# the last two are small epochs (two kernels each)
@pytest.mark.parametrize("m,rows,D,epochs", [(20_000, 20, 50, 1), (20_000, 20, 50, 2), (3_000, 12, 80, 1),
                                             (5_000, 10, 8, 1), (5_000, 10, 8, 2)])
def test_replayed_epochs(cap, m, rows, D, epochs):
    X = GaussianMixture(9 + D, D, 5).rows(0, m)
    W0 = X[draw_initial_rows(4, m, rows * rows)].copy()
    G = dev(oracle.rect_lattice_distances(rows, rows).astype(np.float32))
    # (eager epochs between the replays are a map of their own; with D = 8 a small epoch too)
    G2 = dev(oracle.rect_lattice_distances(7, 7).astype(np.float32))
    Xd, W0d, Wd, W2d = dev(X), dev(W0), dev(W0), dev(W0[:49])

    def call():
        Wd.copy_(W0d)
        for e in range(epochs):
            cap.som.som_epoch(Xd, Wd, G, 2.0 - e, want_stats=False)

    print(f"replayed epochs: m={m} K={rows * rows} D={D} epochs={epochs}", flush=True)
    cap.eager(call)
    want = Wd.cpu().numpy().copy()
    cap.record(call)
    for r in cap.replays(lambda: cap.som.som_epoch(Xd, W2d, G2, 1.0, want_stats=False)):
        # (float64 sums in another order: the float32 weights may differ in their last bit)
        np.testing.assert_allclose(Wd.cpu().numpy(), want, rtol=2e-7, atol=1e-6 * np.abs(want).max(), err_msg=f"replay {r}")
    cap.eager(call)
    np.testing.assert_allclose(Wd.cpu().numpy(), want, rtol=2e-7, atol=1e-6 * np.abs(want).max())


@pytest.mark.parametrize("m,side,D,kind,reproducible,shift", [(20_000, 12, 50, "mst", False, False), (5_000, 9, 100, "rng", False, True),
                                                              (30_000, 66, 40, "rng", False, False), (8_000, 20, 64, "mst", True, True)])
def test_replayed_stages(cap, m, side, D, kind, reproducible, shift):
    """The graph rebuild, the accumulation and the update one by one, on units that are given."""
    K = side * side
    X = GaussianMixture(19 + D, D, 5).rows(0, m)
    W0 = GaussianMixture(20 + D, D, 5).rows(0, K)
    b = np.random.default_rng(D).integers(0, K, size=m).astype(np.int32)
    Xd, W0d, Wd, bd = dev(X), dev(W0), dev(W0), dev(b)
    G = torch.empty((K, K), device="cuda")
    S = torch.empty((K, D), dtype=torch.float64, device="cuda")
    n = torch.empty(K, dtype=torch.int64, device="cuda")
    guarded = torch.empty(1, dtype=torch.int32, device="cuda")
    S2, n2, b2 = torch.empty_like(S[:49]), torch.empty_like(n[:49]), dev(b[:1000] % 49)
    cap.som.som_set_reproducible(reproducible)
    cap.som.som_set_safeguard("shift" if shift else "threshold")

    def call():
        Wd.copy_(W0d)
        cap.som.som_topology(Wd, kind, G=G)
        cap.som.som_accumulate(Xd, bd, K, S, n, zero_first=True)
        cap.som.som_neighborhood_update(S, n, G, 1.5, Wd, n_guarded=guarded)

    print(f"replayed stages: m={m} K={K} D={D} {kind}", flush=True)
    cap.eager(call)
    S_or, n_or = oracle.accumulate(X, None, b, K)
    assert np.array_equal(n.cpu().numpy(), n_or)
    np.testing.assert_allclose(S.cpu().numpy(), S_or, rtol=1e-9, atol=1e-9 * np.abs(X).max() * m)
    want = [t.cpu().numpy().copy() for t in (G, S, n, Wd, guarded)]
    cap.record(call)
    for r in cap.replays(lambda: cap.som.som_accumulate(Xd[:1000], b2, 49, S2, n2, zero_first=True)):
        assert np.array_equal(G.cpu().numpy(), want[0]) and np.array_equal(n.cpu().numpy(), want[2]), f"replay {r}"
        np.testing.assert_allclose(S.cpu().numpy(), want[1], rtol=1e-9, atol=1e-9 * np.abs(X).max() * m, err_msg=f"replay {r}")
        np.testing.assert_allclose(Wd.cpu().numpy(), want[3], rtol=1e-6, atol=1e-6, err_msg=f"replay {r}")
        assert int(guarded.item()) == int(want[4][0])
        for t in (G, S, n, guarded):
            t.fill_(3)
        torch.cuda.synchronize()
