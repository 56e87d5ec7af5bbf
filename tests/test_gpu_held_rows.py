"""The search for rows of 65 to 256 features, which wavefronts hold in registers as half-precision and fp6 parts: the error that
its bound charges per MFMA, and its choices against float64 at the edges of its units, scales and error band."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def som():
    from paper_2604_26555_amd import Som
    s = Som(0)
    yield s
    s.close()


# ------------------------------------------------------------------ what the matrix pipe loses
def significands(rng, shape, bits, ones):
    """Significands of `bits` bits in [1, 2): all ones or random."""
    top = 2 ** (bits - 1)
    return (2.0 - 1.0 / top) * np.ones(shape) if ones else 1.0 + rng.integers(0, top, size=shape) / top


def charge(som, kind, A, Bt, C, units):
    """Largest error of C + A Bt^T in units of 2^-24 (|C| + sum |products|); every sum here is exact in float64 but for the last bits
    of 2^-53, far below a unit."""
    D = som.som_matrix_pipe_probe_parts(kind, torch.from_numpy(A.astype(np.float16)).cuda(), torch.from_numpy(Bt.astype(np.float16)).cuda(),
                                        torch.from_numpy(C.astype(np.float32)).cuda())
    som.som_sync()
    A, Bt, C = A.astype(np.float16).astype(np.float64), Bt.astype(np.float16).astype(np.float64), C.astype(np.float32).astype(np.float64)
    exact = C + np.matmul(A, Bt.transpose(0, 2, 1))
    size = np.abs(C) + np.matmul(np.abs(A), np.abs(Bt).transpose(0, 2, 1))
    worst = float((np.abs(D.cpu().numpy().astype(np.float64) - exact) / (size * U)).max())
    assert worst <= units, worst
    return worst


@pytest.mark.parametrize("kind,bits,K,units", [(0, 11, 16, 16.0), (1, 4, 64, 64.0)])
def test_mfma_accumulation_error_stays_inside_the_charge(som, kind, bits, K, units):
    """The bound charges a half-precision MFMA what seventeen float32 terms can lose in any order of additions (16 units), an fp6
    one what sixty-five can (64).  Sums built against sequential, aligning and truncating adders; values stay normal (the search
    scales the largest element to 2^11 and charges what lies 2^-25 below it apart)."""
    rng = np.random.default_rng(7)
    n, worst = 64, 0.0
    spread, high = (12, 1.0) if kind == 0 else (2, 4.0)     # binades of the format that are used, and its highest
    for ones in (True, False):
        sig = lambda: significands(rng, (n, 32, K), bits, ones)
        sign = lambda: rng.choice([-1.0, 1.0], size=(n, 32, K))
        # same-sign products below half a unit of C's last place; C of either sign
        for depth in (22, 24, 26):
            for c in (1.0, -1.0):
                C = c * 2.0 ** depth * (1.0 + rng.integers(0, 2 ** 23, size=(n, 32, 32)) / 2.0 ** 23)
                worst = max(worst, charge(som, kind, sig(), sig(), C, units))
        # descending exponents, a dominant product, cancellation against C, random exponents
        down = high * 2.0 ** -(np.arange(K) % (spread + 1))
        one = high * np.where(np.arange(K) == K // 2, 1.0, 2.0 ** -spread)
        wide = lambda: high * 2.0 ** -rng.integers(0, spread + 1, size=(n, 32, K))
        for A in (sig() * down, sig() * one * sign(), sig() * wide() * sign()):
            A = np.take_along_axis(A, np.argsort(rng.random((n, 1, K)), axis=2).repeat(32, axis=1), axis=2)
            B = sig() * wide()
            s = np.matmul(A, B.transpose(0, 2, 1))
            for C in (0 * s, -s * (1.0 + 1e-3 * rng.normal(size=s.shape)), rng.uniform(-1, 1, size=s.shape) * 2.0 ** 8):
                worst = max(worst, charge(som, kind, A, B, C, units))
    print(f"kind {kind}: largest error {worst:.2f} units, charged {units}", flush=True)


# ------------------------------------------------------------------ choices against float64
def check(som, X, W, idx=None):
    """The chosen node is as near as the nearest one, to within what float32 direct differences resolve: a sum of D squares of
    rounded differences errs by at most (D + 3) 2^-24 of itself, on either side."""
    b, _, _ = som.som_bmu(X, W, idx=idx)
    rows = X if idx is None else X[idx.long()]
    w = W.double()
    for lo in range(0, rows.shape[0], 1024):
        x = rows[lo:lo + 1024].double()
        d2 = torch.stack([((x - w[k]) ** 2).sum(1) for k in range(w.shape[0])], 1) if w.shape[0] < 64 else \
            ((x[:, None, :] - w[None, :, :]) ** 2).sum(2)
        got = d2.gather(1, b[lo:lo + 1024].long()[:, None])[:, 0]
        excess = (got / d2.min(1).values.clamp_min(1e-300) - 1.0).max().item()
        assert excess <= (X.shape[1] + 4) * 2.0 ** -23, (lo, excess)


def draw(m, K, D, seed, noise=0.3):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((m, D), device="cuda", generator=g)
    W = X[torch.randint(m, (K,), device="cuda", generator=g)] + noise * torch.randn((K, D), device="cuda", generator=g)
    return X, W.contiguous()


@pytest.mark.parametrize("D", [65, 68, 80, 81, 96, 97, 99, 128, 129, 160, 161, 192, 193, 200, 224, 225, 240, 241, 255, 256])
def test_units_and_tiles(som, D):
    """Rows that end anywhere in a unit of 32 features, maps that end anywhere in a block of 32 or a stage of 128 nodes, tiles that
    are not full, one block, two and an odd number of them; the sizes where several workgroups share a tile's nodes, and where not."""
    for m, K in ((1, 2), (127, 31), (128, 33), (129, 64), (300, 97), (1000, 129), (600, 333)):
        check(som, *draw(m, K, D, D + m))
    g = torch.Generator(device="cuda").manual_seed(D)
    X, W = draw(900, 70, D, D)
    big = torch.randn((900, D + 3), device="cuda", generator=g)              # rows that start anywhere, and a list of rows
    big[:, 1:D + 1] = X
    idx = torch.randint(900, (700,), device="cuda", generator=g).int()
    check(som, big[:, 1:D + 1], W, idx)


@pytest.mark.parametrize("D", [70, 200, 256])
def test_error_band(som, D):
    """Nodes in pairs so close that the samples' best two scores lie on both sides of the error band, and triples within one class:
    a bound that is too small decides some of them by scores that are wrong."""
    for gap in (1e-1, 1e-2, 1e-3, 1e-4, 1e-5):
        g = torch.Generator(device="cuda").manual_seed(D)
        base = torch.randn((60, D), device="cuda", generator=g)
        W = torch.cat([base, base + gap * torch.randn((60, D), device="cuda", generator=g), base[:40] + gap * torch.randn((40, D), device="cuda", generator=g)])
        X = W[torch.randint(160, (6000,), device="cuda", generator=g)] + 0.5 * torch.randn((6000, D), device="cuda", generator=g)
        check(som, X, W.contiguous())


@pytest.mark.parametrize("D", [100, 224])
def test_scales(som, D):
    """A sample is scaled by its own largest element, the weights by theirs: samples far outside the map's spread and far inside it,
    up to and beyond the largest difference of the scales, features of very different size, values near the ends of float32, maps
    that have collapsed, weights that are all the same."""
    X, W = draw(500, 90, D, 3)
    for s in (1e-17, 1e-8, 1e8, 1e17):
        check(som, X * s, (W * s).contiguous())
    for s in (1e-12, 1e-9, 1e-6, 1e-3, 1e3):
        check(som, X, (W * s).contiguous())
        check(som, X * s, W)
    cols = torch.logspace(-6, 6, D, device="cuda")
    check(som, X * cols, (W * cols).contiguous())
    check(som, X + 1000.0, (W + 1000.0).contiguous())
    b, _, _ = som.som_bmu(X, W[:1].expand(90, D).contiguous())               # all as near: the lowest index
    assert (b == 0).all()


@pytest.mark.parametrize("D", [66, 256])
def test_rows_that_hold_no_numbers(som, D):
    """NaN and infinite values in rows and in weights: such samples go to the all-nodes pass, the others are not touched by them."""
    X, W = draw(700, 140, D, 4)
    clean, _, _ = som.som_bmu(X, W)
    Y = X.clone()
    Y[::7, D - 1] = float("nan")
    Y[3::7, 0] = float("inf")
    b, _, _ = som.som_bmu(Y, W)
    keep = torch.isfinite(Y).all(1)
    assert (b[keep] == clean[keep]).all() and ((b >= 0) & (b < 140)).all()
    V = W.clone()
    V[17, 5] = float("nan")
    b, _, _ = som.som_bmu(X, V)
    keep = clean != 17
    assert (b[keep] == clean[keep]).all() and (b != 17).all()
