"""The work that programs on this library give it, as cases that can be timed: what a case holds, how its inputs are
made, one pass through the public entry points, and the bytes and operations that pass cannot do without.

Sizes are those of the synthetic workloads in ``synth/configs.py``, of the feature and grid axes of ``bench.py
--workload scale`` and of the tests, or odd ones in the same ranges.  Inputs are drawn on the GPU from the seed alone:
Gaussian mixtures (centres uniform in [-10, 10]^D, per-axis deviations uniform in [0.2, 3]) or the uniform [0, 1)
matrices of the speed axes.  The weights are those of a map in the middle of its training: a few batch epochs in plain
torch on a sample of the rows, with the radius falling to the case's own.
"""
import math

import torch

import paper_2604_26555_amd as pkg

DEVICE = "cuda:0"
SAMPLE = 16384          # rows that the weights are warmed up on
BLOCK = 1 << 20         # rows made at a time

# Fields of a case:
#   kind      train    a whole short training from initial rows, `epochs` epochs with the radius falling from 10 sigma to sigma
#             epoch    one epoch of a lattice map on resident rows
#             graph    one epoch of a data-driven map: graph rebuilt from the weights, then the epoch
#             project  best-matching units of rows under fixed weights
#             stages   search, accumulation and update called one by one, with learning rate and momentum
#             host     one epoch on rows in ordinary host memory, streamed in chunks
#   n, d      rows and features;  rows, cols: the map's sides (K = rows * cols);  topology: rect, hex, mst or rng
#   sigma     radius of the epoch;  listed: rows presented through a row list (0: all rows);  data: mixture or uniform
#   stats     the epoch's statistics (quantisation error) are asked for, as a program that logs its progress does;
#             for project: the distances and the quantisation error are
#   fixed     fixed order of summation (reproducible sums);  shift: the shifted-exponent safeguard


def _case(name, kind, n, d, rows, cols, topology, sigma, listed=0, stats=False, data="mixture", epochs=1, chunk=0,
          fixed=False, shift=False):
    c = dict(kind=kind, n=int(n), d=int(d), rows=int(rows), cols=int(cols), topology=topology, sigma=float(sigma),
             listed=int(listed), stats=bool(stats), data=data, epochs=int(epochs), chunk=int(chunk), fixed=bool(fixed),
             shift=bool(shift))
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # new observations looked up on a trained map, a thousand at a time: all latency
        _case("project_1k", "project", 1000, 50, 32, 32, "hex", 1.0, stats=True),
        # a whole training of a small map on a small table (cfg0): ten epochs back to back
        _case("train_10k_d8", "train", 10_000, 8, 10, 10, "rect", 0.5, epochs=10),
        # an ordinary table of odd sizes on a map that fills no block; the quantisation error is logged every epoch
        _case("epoch_250k_d37_stats", "epoch", 250_013, 37, 19, 23, "rect", 3.0, stats=True),
        # the headline workload (cfg1)
        _case("epoch_1m_d50", "epoch", 1_000_000, 50, 32, 32, "hex", 4.0),
        # the largest map of the grid axis
        _case("epoch_1m_k4096", "epoch", 1_000_000, 50, 64, 64, "rect", 6.0),
        # the feature axis: wide rows and very wide ones
        _case("epoch_1m_d200", "epoch", 1_000_000, 200, 32, 32, "hex", 4.0, data="uniform"),
        _case("epoch_100k_d2000", "epoch", 100_000, 2000, 32, 32, "hex", 4.0, data="uniform"),
        # spanning-tree map, graph rebuilt every epoch (cfg2)
        _case("mst_10m_d50", "graph", 10_000_000, 50, 32, 32, "mst", 4.0),
        # neighbourhood-graph map, a tenth of the rows drawn for every epoch through a sorted row list (cfg3)
        _case("rng_subset_4m_of_40m", "graph", 40_000_000, 50, 32, 32, "rng", 3.0, listed=4_000_000),
        # holdout rows (30 % of the table, a row list) projected with distances and quantisation error
        _case("holdout_900k_d25", "project", 3_000_000, 25, 20, 20, "hex", 1.0, listed=900_000, stats=True),
        # the three stages one by one with momentum, the shifted safeguard and reproducible sums
        _case("stages_500k_d64_fixed", "stages", 500_000, 64, 20, 20, "rect", 2.0, fixed=True, shift=True),
        # rows in ordinary host memory in chunks (cfg4's regime)
        _case("host_4m_d50", "host", 4_000_000, 50, 32, 32, "rect", 4.0, chunk=250_000, stats=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "epoch", "epoch", "epoch", "wide", "graph", "subset", "project", "holdout", "stages", "host"])
    rows = _log(rng, 8, 64)
    cols = max(8, min(64, int(round(rows * rng.uniform(0.7, 1.4)))))
    d = _log(rng, 4, 64)
    k = rows * cols
    lattice = rng.choice(["rect", "hex"])
    sigma = round(rng.uniform(0.5, min(rows, cols) / 3.0), 2)
    if kind == "train":
        rows = cols = rng.randint(8, 16)
        return _case(None, "train", _log(rng, 2_000, 100_000), rng.randint(4, 24), rows, cols, lattice, 0.5, epochs=rng.randint(5, 12))
    if kind == "wide":
        rows, cols = rng.randint(12, 36), rng.randint(12, 36)
        d = _log(rng, 65, 2000)
        n = min(_log(rng, 10_000, 1_000_000), int(2e8) // d)
        return _case(None, "epoch", n, d, rows, cols, lattice, round(rng.uniform(1.0, 4.0), 2), data="uniform")
    most = int(min(10_000_000, 5.1e11 / (k * d)))                  # never more work than the largest listed case
    if kind == "epoch":
        return _case(None, "epoch", _log(rng, 20_000, most), d, rows, cols, lattice, sigma, stats=rng.random() < 0.3,
                     data=rng.choice(["mixture", "mixture", "uniform"]))
    if kind in ("graph", "subset"):
        n = _log(rng, 50_000, most)
        big = min(10 * n, int(2e9) // d) if kind == "subset" else n
        return _case(None, "graph", big, d, rows, cols, rng.choice(["mst", "rng"]), min(sigma, 8.0), listed=n if big > n else 0,
                     stats=rng.random() < 0.3)
    if kind == "project":
        return _case(None, "project", _log(rng, 200, 200_000), d, rows, cols, lattice, 1.0, stats=rng.random() < 0.7)
    if kind == "holdout":
        n = _log(rng, 100_000, min(most, 4_000_000))
        return _case(None, "project", n, d, rows, cols, lattice, 1.0, listed=max(1, int(0.3 * n)), stats=True)
    if kind == "stages":
        rows, cols = rng.randint(8, 32), rng.randint(8, 32)
        return _case(None, "stages", _log(rng, 20_000, min(int(5.1e11 / (rows * cols * d)), 2_000_000)), d, rows, cols, lattice,
                     round(rng.uniform(1.0, 4.0), 2), fixed=rng.random() < 0.5, shift=rng.random() < 0.5)
    n = _log(rng, 100_000, int(2e8) // max(d, 16))
    n = min(n, most)
    return _case(None, "host", n, d, rows, cols, lattice, sigma, chunk=max(4096, n // rng.randint(4, 16)), stats=True)


def _rows(case, gen):
    n, d = case["n"], case["d"]
    X = torch.empty((n, d), device=DEVICE)
    if case["data"] == "uniform":
        for lo in range(0, n, BLOCK):
            X[lo:lo + BLOCK].uniform_(generator=gen)
        return X
    comps = 20
    centres = torch.empty((comps, d), device=DEVICE).uniform_(-10, 10, generator=gen)
    std = torch.empty((comps, d), device=DEVICE).uniform_(0.2, 3, generator=gen)
    # unequal components, and 5 % of background for the graph maps
    edges = torch.empty(comps, device=DEVICE).exponential_(generator=gen) + 0.05
    edges = torch.cumsum(edges / edges.sum(), 0)
    noise = 0.05 if case["kind"] == "graph" else 0.0
    for lo in range(0, n, BLOCK):
        out = X[lo:lo + BLOCK]
        m = out.shape[0]
        comp = torch.searchsorted(edges, torch.rand(m, device=DEVICE, generator=gen)).clamp_(max=comps - 1)
        torch.randn((m, d), device=DEVICE, generator=gen, out=out)
        out.mul_(std[comp]).add_(centres[comp])
        if noise:
            back = torch.rand(m, device=DEVICE, generator=gen) < noise
            out.copy_(torch.where(back[:, None], torch.empty_like(out).uniform_(-15, 15, generator=gen), out))
    return X


def _lattice(case):
    kind = case["topology"] if case["topology"] in ("rect", "hex") else "rect"
    return torch.from_numpy(pkg.topology.lattice_distances(case["rows"], case["cols"], kind)).to(DEVICE)


def _warm_weights(case, X, gen):
    """Weights of a map in the middle of its training (plain torch in float64, matrix products only)."""
    k = case["rows"] * case["cols"]
    Xs = X[:SAMPLE].double()
    W = Xs[torch.randperm(Xs.shape[0], device=DEVICE, generator=gen)[:k]] if Xs.shape[0] >= k else \
        Xs[torch.randint(Xs.shape[0], (k,), device=DEVICE, generator=gen)] + 0.1 * torch.randn((k, case["d"]), device=DEVICE, generator=gen)
    if case["kind"] == "train":
        return W.float().contiguous()
    if case["topology"] == "mst":                      # a chain is a tree: nodes close together along a path
        place = torch.arange(k, device=DEVICE, dtype=torch.float64)
        G = (place[:, None] - place[None, :]).abs()
    else:
        G = _lattice(case).double()
    for factor in (4.0, 2.5, 1.5, 1.0):
        h = torch.exp(-G * G / (2.0 * (factor * case["sigma"]) ** 2))
        best = (Xs @ W.t() - 0.5 * (W * W).sum(1)).argmax(1)
        hit = torch.zeros((Xs.shape[0], k), device=DEVICE, dtype=torch.float64)
        hit.scatter_(1, best[:, None], 1.0)
        hit_h = hit @ h
        den = hit_h.sum(0)[:, None]
        W = torch.where(den > 1e-30, (hit_h.t() @ Xs) / den.clamp_min(1e-30), W)
    return W.float().contiguous()


_contexts = {}


def _context(case):
    """The program's library context: one for each set of options, kept.  The update rule with momentum, whose velocity
    buffer has the map's size, stays on contexts of its own."""
    key = (case["fixed"], case["shift"], case["kind"] == "stages")
    if key not in _contexts:
        som = pkg.Som(0)
        som.som_set_reproducible(case["fixed"])
        som.som_set_safeguard("shift" if case["shift"] else "threshold")
        _contexts[key] = som
    return _contexts[key]


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    X = _rows(case, gen)
    s = dict(case=case, som=_context(case), X=X, W0=_warm_weights(case, X, gen), idx=None)
    k, d = case["rows"] * case["cols"], case["d"]
    if case["kind"] != "project":
        s["G"] = torch.empty((k, k), device=DEVICE) if case["kind"] == "graph" else _lattice(case)
    if case["listed"]:
        # a sorted list of distinct rows: one drawn from every stretch of n // listed
        m, stretch = case["listed"], case["n"] // case["listed"]
        s["idx"] = (torch.arange(m, device=DEVICE) * stretch +
                    torch.randint(stretch, (m,), device=DEVICE, generator=gen)).int()
    if case["kind"] == "stages":
        s["S"] = torch.empty((k, d), device=DEVICE, dtype=torch.float64)
        s["count"] = torch.empty(k, device=DEVICE, dtype=torch.int64)
        s["velocity0"] = 0.01 * torch.randn((k, d), device=DEVICE, generator=gen)
    if case["kind"] == "project":
        m = case["listed"] or case["n"]
        s["d2"] = torch.empty(m, device=DEVICE) if case["stats"] else None
        s["qe"] = torch.empty(2, device=DEVICE, dtype=torch.float64) if case["stats"] else None
    if case["kind"] == "host":
        s["X"] = X.cpu().numpy()
    return s


def _statistics(st):
    return [] if st is None else [st.sum_dist, st.sum_dist2]


def run(s):
    case, som, X = s["case"], s["som"], s["X"]
    kind = case["kind"]
    if kind == "project":
        bmu, d2, qe = som.som_bmu(X, s["W0"], idx=s["idx"], d2=s["d2"], qe=s["qe"])
        return [bmu] if d2 is None else [bmu, d2, qe]
    W = s["W0"].clone()                                   # the weights are trained in place
    if kind == "train":
        for e in range(case["epochs"]):
            fall = 1.0 - e / max(1, case["epochs"] - 1)
            som.som_epoch(X, W, s["G"], case["sigma"] * (1.0 + 9.0 * fall), want_stats=False)
        return [W]
    if kind == "epoch":
        return [W] + _statistics(som.som_epoch(X, W, s["G"], case["sigma"], want_stats=case["stats"]))
    if kind == "graph":
        som.som_topology(W, case["topology"], G=s["G"])
        st = som.som_epoch(X, W, s["G"], case["sigma"], idx=s["idx"], want_stats=case["stats"])
        return [W, s["G"]] + _statistics(st)
    if kind == "stages":
        velocity = s["velocity0"].clone()
        som.som_set_update_rule(0.8, 0.5, velocity)
        bmu, _, _ = som.som_bmu(X, W)
        som.som_accumulate(X, bmu, W.shape[0], s["S"], s["count"])
        som.som_neighborhood_update(s["S"], s["count"], s["G"], case["sigma"], W)
        return [bmu, s["S"], s["count"], W, velocity]
    return [W] + _statistics(som.som_epoch_host(X, W, s["G"], case["sigma"], case["chunk"]))


def work(case):
    n, d, k = case["n"], case["d"], case["rows"] * case["cols"]
    m = case["listed"] or n
    w, g = 4.0 * k * d, 4.0 * k * k
    nbytes = 4.0 * m * d + w + (4.0 * m if case["listed"] else 0.0)
    flops = 2.0 * m * k * d
    if case["kind"] == "project":
        return {"bytes": nbytes + (8.0 if case["stats"] else 4.0) * m, "flops": flops}
    nbytes += w + g                                          # the weights go back, the node distances come in
    flops += m * d + 2.0 * k * k * (d + 1)
    if case["kind"] == "graph":
        flops += 3.0 * k * k * d
    if case["kind"] == "stages":
        nbytes += 4.0 * m + 8.0 * k * (d + 1) + 2.0 * w
    return {"bytes": nbytes, "flops": flops * case["epochs"]}


def tolerance(case):
    # Float32 direct differences decide between nodes that are equally near to within a few 2^-24, so a handful of
    # samples in a million may go to the other node; sums are float64 and weights are rounded to float32 once.
    if case["kind"] == "project":
        return {"rel": 1e-5, "differ": 1e-3}
    if case["kind"] == "stages":
        return {"rel": 1e-4, "differ": 1e-2}
    return {"rel": 1e-4}
