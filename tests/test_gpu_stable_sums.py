"""Sums in a fixed order: ranks of samples among those of the same node, at numbers of nodes on both sides of a power of two."""
import pytest
import torch

pkg = pytest.importorskip("paper_2604_26555_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 3, 63, 64, 65, 255, 256, 257, 1023, 1025, 8191, 8192])
def test_fixed_order_sums(K):
    """Nodes spread evenly, all samples on one node, neighbours in pairs, and samples of no node; blocks that end inside a wavefront.  Integers
    add up without rounding, so the sums are exact whatever the order, and two calls agree in every bit on other values."""
    som = pkg.Som(0)
    som.som_set_reproducible(True)
    g = torch.Generator(device="cuda").manual_seed(K)
    for m in (1, 65, 1000, 70_001):
        X = torch.randint(-1000, 1000, (m, 20), device="cuda", generator=g).float()
        for kind in range(4):
            b = torch.randint(K, (m,), device="cuda", generator=g)
            if kind == 1:
                b[:] = K - 1
            elif kind == 2:
                b = (torch.arange(m, device="cuda") // 2) % K
            elif kind == 3:
                b[::3] = -1
                b[1::5] = K
            b = b.int()
            S = torch.empty((K, 20), device="cuda", dtype=torch.float64)
            n = torch.empty(K, device="cuda", dtype=torch.int64)
            som.som_accumulate(X, b, K, S, n)
            on = (b >= 0) & (b < K)
            want = torch.zeros((K, 20), dtype=torch.float64).index_add_(0, b[on].cpu().long(), X[on].cpu().double())
            assert torch.equal(S.cpu(), want)
            assert torch.equal(n.cpu(), torch.bincount(b[on].cpu().long(), minlength=K))
            Y = torch.randn((m, 20), device="cuda", generator=g)
            som.som_accumulate(Y, b, K, S, n)
            T = torch.empty_like(S)
            som.som_accumulate(Y, b, K, T, n)
            assert torch.equal(S, T)
