"""The statistics of an epoch: sums that no earlier call has left anything in, and times from the device's clock."""
import time

import pytest
import torch

pkg = pytest.importorskip("paper_2604_26555_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("search", ["auto", "float32"])
@pytest.mark.parametrize("m,D,K", [(1, 5, 3), (300, 2, 40), (5000, 8, 100), (20_001, 37, 437), (9000, 64, 130), (3000, 100, 200), (2500, 300, 350)])
def test_epoch_statistics(search, m, D, K):
    """Resident and streamed epochs, and look-ups between them, give the same sums however they follow each other: float64 sums of
    the same float32 distances, in orders of their own (m additions of 2^-53 at most)."""
    som = pkg.Som(0)
    som.som_set_search(search)
    g = torch.Generator(device="cuda").manual_seed(m + D)
    X = torch.randn((m, D), device="cuda", generator=g)
    W = torch.randn((K, D), device="cuda", generator=g)
    side = torch.arange(K, device="cuda", dtype=torch.float32)
    G = (side[:, None] - side[None, :]).abs()
    qe = torch.empty(2, device="cuda", dtype=torch.float64)
    seen = []
    for _ in range(2):
        for shift in (False, True):
            som.som_set_safeguard("shift" if shift else "threshold")
            t0 = time.perf_counter()
            st = som.som_epoch(X, W.clone(), G, 3.0)
            wall = 1e3 * (time.perf_counter() - t0)
            assert 0.0 < st.ms_bmu_acc < wall and 0.0 < st.ms_update < wall and st.m == m
            seen.append((st.sum_dist, st.sum_dist2, st.n_recheck, st.n_empty, st.n_guarded))
            som.som_bmu(X, W, d2=torch.empty(m, device="cuda"), qe=qe)
            st = som.som_epoch_host(X.cpu().numpy(), W.clone(), G, 3.0, max(1, m // 3))
            assert st.ms_bmu_acc > 0.0 and st.ms_update > 0.0
            seen.append((st.sum_dist, st.sum_dist2, st.n_recheck, st.n_empty, st.n_guarded))
    for s in seen:
        assert abs(s[0] / seen[0][0] - 1.0) <= m * 2.0 ** -52 and abs(s[1] / seen[0][1] - 1.0) <= m * 2.0 ** -52
        assert s[2:4] == seen[0][2:4]
    assert abs(qe[0].item() / seen[0][0] - 1.0) <= 1e-6
