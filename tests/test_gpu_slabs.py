"""Sums by LDS atomics: nodes dealt out to slabs, at numbers of nodes around each number of slabs."""
import pytest
import torch

pkg = pytest.importorskip("paper_2604_26555_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [7, 31, 50, 63])
@pytest.mark.parametrize("slabs", [1, 2, 3, 5, 9, 16])
def test_nodes_of_every_slab(D, slabs):
    """Integers add up without rounding, so the sums are exact whatever the order: nodes in turn, a crowd on the last node, samples of no node."""
    som = pkg.Som(0)
    most = 150 * 1024 // (8 * (D + 1))                      # nodes of a slab
    g = torch.Generator(device="cuda").manual_seed(D + slabs)
    for K in (most * slabs, most * slabs - 1, most * (slabs - 1) + 1):
        m = 40_000 + slabs
        X = torch.randint(-1000, 1000, (m, D), device="cuda", generator=g).float()
        b = (torch.arange(m, device="cuda") * 7) % K
        b[::5] = K - 1
        b[::11] = -1
        b[1::13] = K
        rows = torch.randint(m, (m - 100,), device="cuda", generator=g).int()
        for idx in (None, rows):
            use, x = (b, X) if idx is None else (b[100:], X[rows.long()])
            S = torch.empty((K, D), device="cuda", dtype=torch.float64)
            n = torch.empty(K, device="cuda", dtype=torch.int64)
            som.som_accumulate(X, use.int(), K, S, n, idx=idx)
            on = (use >= 0) & (use < K)
            want = torch.zeros((K, D), dtype=torch.float64).index_add_(0, use[on].cpu(), x[on].cpu().double())
            assert torch.equal(S.cpu(), want)
            assert torch.equal(n.cpu(), torch.bincount(use[on].cpu(), minlength=K))


def test_two_slabs_of_narrow_rows_cost_little_more_than_one():
    """4096 nodes of three features fit one slab, of four two: 1.6 times as long a call when a slab left LDS a row a wavefront, 0.8 a lane a cell."""
    som = pkg.Som(0)
    m, K, times = 20_000, 4096, []
    for D in (3, 4):
        X = torch.ones((m, D), device="cuda")
        b = (torch.arange(m, device="cuda") % K).int()
        S, n = torch.empty((K, D), device="cuda", dtype=torch.float64), torch.empty(K, device="cuda", dtype=torch.int64)
        best = float("inf")
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(50):
                som.som_accumulate(X, b, K, S, n)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) / 50)
        times.append(best * 1e3)
    print(f"three features {times[0]:.1f} us, four {times[1]:.1f}", flush=True)
    assert times[1] < 1.25 * times[0], times
