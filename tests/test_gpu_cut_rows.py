"""The search for rows of more than 256 features on maps of more than 320 nodes, whose samples are cut once beforehand: its choices
against float64 at the edges of its chunks, stages, tiles, pieces and passes, and of its line to the tile that serves smaller maps."""
import pytest
import torch

from test_gpu_held_rows import check, draw, som  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [257, 258, 260, 287, 288, 289, 319, 320, 321, 383, 385, 450, 513])
def test_chunks_and_stages(som, D):  # noqa: F811
    """Rows that end anywhere in a unit of 32 features or a chunk of 64, maps that end anywhere in a block of 32, a stage of 64 or a tile of
    256 nodes (one, two, three or four stages of the last one), tiles of 256 samples that are not full."""
    for m, K in ((1, 321), (31, 352), (255, 384), (257, 385), (300, 449), (513, 512), (600, 577)):
        check(som, *draw(m, K, D, D + m))


@pytest.mark.parametrize("K", [256, 257, 320, 321])
def test_both_sides_of_the_line_to_the_tile(som, K):  # noqa: F811
    for D in (256, 257, 300):
        check(som, *draw(700, K, D, K))


@pytest.mark.parametrize("m,K", [(33000, 330), (66000, 400), (70000, 1024), (1000, 4100)])
def test_pieces(som, m, K):  # noqa: F811
    """Whole rounds of tiles and a last, partial one, in pieces as large and in smaller ones; few rows in pieces of eight stages; the first and the last
    rows of each."""
    X, W = draw(m, K, 260, m)
    rows = torch.cat([torch.arange(0, min(m, 512)), torch.arange(max(0, m - 1024), m), torch.randint(m, (1024,))]).cuda()
    b, _, _ = som.som_bmu(X, W)
    x, w = X[rows].double(), W.double()
    for lo in range(0, len(rows), 64):
        d2 = ((x[lo:lo + 64, None, :] - w[None, :, :]) ** 2).sum(2)
        got = d2.gather(1, b[rows[lo:lo + 64]].long()[:, None])[:, 0]
        assert (got / d2.min(1).values - 1.0).max().item() <= 264 * 2.0 ** -23


@pytest.mark.parametrize("m,K,line", [(50_000, 600, 43_008), (22_526, 1024, 16_384), (100_000, 1024, 98_304), (50_497, 800, 49_152), (100_000, 1600, 98_304)])
def test_whole_rounds_and_smaller_pieces_behind_them(som, m, K, line):  # noqa: F811
    """Whole rounds of workgroups end at row `line`; the rows behind it are searched in pieces of four stages (as the others), two, one, one, and
    two where the others take eight.  Nodes in close pairs, so that winners of every place decide; rows on both sides of the line and at either end."""
    X, W = draw(m, K, 260, m + K)
    W[K // 2:] = W[:K - K // 2] + 1e-4 * torch.randn((K - K // 2, 260), device="cuda", generator=torch.Generator(device="cuda").manual_seed(K))
    rows = torch.cat([torch.arange(0, 512), torch.arange(line - 512, line + 512), torch.arange(m - 512, m), torch.randint(line, m, (1024,))]).cuda()
    b, _, _ = som.som_bmu(X, W)
    x, w = X[rows].double(), W.double()
    for lo in range(0, len(rows), 64):
        d2 = ((x[lo:lo + 64, None, :] - w[None, :, :]) ** 2).sum(2)
        got = d2.gather(1, b[rows[lo:lo + 64]].long()[:, None])[:, 0]
        assert (got / d2.min(1).values - 1.0).max().item() <= 264 * 2.0 ** -23


def test_lists_of_rows_and_rows_that_start_anywhere(som):  # noqa: F811
    X, W = draw(900, 350, 301, 1)
    big = torch.randn((900, 305), device="cuda")
    big[:, 1:302] = X
    idx = torch.randint(900, (700,), device="cuda").int()
    check(som, big[:, 1:302], W, idx)


@pytest.mark.parametrize("K", [320, 321, 448, 449, 512, 513])
@pytest.mark.parametrize("m", [129_000, 131_072, 140_000])
def test_both_sides_of_the_line_by_rows(som, m, K):  # noqa: F811
    """Rows that fill the tile's rounds, and rows that just do not; the first and the last ones."""
    X, W = draw(m, K, 260, m + K)
    rows = torch.cat([torch.arange(0, 512), torch.arange(m - 1024, m), torch.randint(m, (1024,))]).cuda()
    b, _, _ = som.som_bmu(X, W)
    x, w = X[rows].double(), W.double()
    for lo in range(0, len(rows), 64):
        d2 = ((x[lo:lo + 64, None, :] - w[None, :, :]) ** 2).sum(2)
        got = d2.gather(1, b[rows[lo:lo + 64]].long()[:, None])[:, 0]
        assert (got / d2.min(1).values - 1.0).max().item() <= 264 * 2.0 ** -23


@pytest.mark.parametrize("m", [32768, 40001])
def test_long_lists(som, m):  # noqa: F811
    """Six nodes close together everywhere, so that almost every row is listed: as many blocks of the list as workgroups cut them, and more; the
    first and the last rows."""
    g = torch.Generator(device="cuda").manual_seed(m)
    base = torch.randn((60, 260), device="cuda", generator=g)
    W = (base[:, None, :] + 1e-4 * torch.randn((60, 6, 260), device="cuda", generator=g)).reshape(360, 260)
    X = torch.randn((m + 7, 260), device="cuda", generator=g)
    idx = torch.randperm(m + 7, device="cuda", generator=g)[:m].int()
    b, _, _ = som.som_bmu(X, W, idx=idx)
    rows = torch.cat([torch.arange(0, 600), torch.arange(m - 1500, m), torch.randint(m, (1000,))]).cuda()
    x, w = X[idx[rows].long()].double(), W.double()
    for lo in range(0, len(rows), 100):
        d2 = ((x[lo:lo + 100, None, :] - w[None, :, :]) ** 2).sum(2)
        got = d2.gather(1, b[rows[lo:lo + 100]].long()[:, None])[:, 0]
        assert (got / d2.min(1).values - 1.0).max().item() <= 264 * 2.0 ** -23


@pytest.mark.parametrize("D", [300, 512])
def test_error_band(som, D):  # noqa: F811
    """Pairs and triples of nodes so close that the samples' best two scores lie on both sides of the error band: lists of any length, short ones
    (candidates stage by stage) and long ones (tile by tile), and records that overflow."""
    for gap in (1e-1, 1e-2, 1e-3, 1e-4, 1e-5):
        g = torch.Generator(device="cuda").manual_seed(D)
        base = torch.randn((150, D), device="cuda", generator=g)
        W = torch.cat([base, base + gap * torch.randn((150, D), device="cuda", generator=g), base[:60] + gap * torch.randn((60, D), device="cuda", generator=g)])
        X = W[torch.randint(360, (3000,), device="cuda", generator=g)] + 0.5 * torch.randn((3000, D), device="cuda", generator=g)
        check(som, X, W.contiguous())
    W = base[:1] + 1e-6 * torch.randn((360, D), device="cuda", generator=g)
    check(som, X[:1500], W.contiguous())


def test_scales(som):  # noqa: F811
    """Each chunk of a sample is scaled by its own largest element: features of very different size, samples far outside the map's
    spread and far inside it, values near the ends of float32, weights that are all the same."""
    D = 330
    X, W = draw(400, 340, D, 3)
    for s in (1e-17, 1e-8, 1e8, 1e17):
        check(som, X * s, (W * s).contiguous())
    for s in (1e-12, 1e-6, 1e3):
        check(som, X, (W * s).contiguous())
        check(som, X * s, W)
    cols = torch.logspace(-6, 6, D, device="cuda")
    check(som, X * cols, (W * cols).contiguous())
    cols = torch.where(torch.arange(D, device="cuda") < 64, 0.0, 1.0)        # a chunk of zeros
    check(som, X * cols, (W * cols).contiguous())
    check(som, X + 1000.0, (W + 1000.0).contiguous())
    b, _, _ = som.som_bmu(X, W[:1].expand(340, D).contiguous())              # all as near: the lowest index
    assert (b == 0).all()


def test_rows_that_hold_no_numbers(som):  # noqa: F811
    X, W = draw(700, 340, 270, 4)
    clean, _, _ = som.som_bmu(X, W)
    Y = X.clone()
    Y[::7, 269] = float("nan")
    Y[3::7, 0] = float("inf")
    b, _, _ = som.som_bmu(Y, W)
    keep = torch.isfinite(Y).all(1)
    assert (b[keep] == clean[keep]).all() and ((b >= 0) & (b < 340)).all()
    V = W.clone()
    V[17, 5] = float("nan")
    b, _, _ = som.som_bmu(X, V)
    keep = clean != 17
    assert (b[keep] == clean[keep]).all() and (b != 17).all()
