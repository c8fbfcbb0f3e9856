"""Workloads of the walk library for timing: what its users run, small to large.

Each case is a graph, a walk and the entry point that runs it.  The graphs are
the kinds the library is built for: R-MAT graphs with (a, b, c) = (.57, .19,
.19) and Chung-Lu graphs of exponent 2.1, symmetrised, without self-loops and
repeated edges, ids shuffled, rows sorted; integer edge weights uniform in
[1, 255] or Zipf(1.2) clipped to 65535, the same in both directions of an edge;
labels uniform in {0..4}.  Start vertices are drawn uniformly (isolated
vertices among them, whose walks end at once), or all are the vertex of
largest degree (personalised PageRank).  Everything comes from the seed alone.

Every result is whole numbers: vertex ids, 0xFFFFFFFF after an early end.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2404_08364_amd import flowwalk as fw

MASK = (1 << 64) - 1
SCHEMA = (0, 1, 2, 3, 4)
STOP = (1, 5)
FACTORS = (1, 2, 4)  # node2vec p = 2, q = 1/2
# zeta(1.2): Zipf's mass over all positive integers, the clipped ones included.
ZETA_1_2 = 5.591582441177751


def _case(name, **kw):
    base = dict(entry="walk", graph="rmat", scale=20, edge_factor=16, weights="uniform",
                labels=False, algo="node2vec", n=1, length=80, starts="uniform")
    base.update(kw)
    if name:
        base["name"] = name
    return base


def listed():
    return [
        # A single user's lookup on a small graph: a handful of walks, where
        # the launch and the chain of dependent hops are all there is.
        _case("n2v_tiny", scale=12, edge_factor=8, n=16, length=20),
        # A few recommendations' walks on a graph with hubs: too few queries
        # to fill the chip.
        _case("deepwalk_few", algo="deepwalk", n=33),
        # A training mini-batch of starts: a few thousand node2vec walks.
        _case("n2v_batch", n=3001),
        # One epoch's share of a node2vec corpus on the benchmark's graph.
        _case("n2v_large", scale=22, weights="zipf", n=524288),
        # The same without edge weights, as most published node2vec graphs are.
        _case("n2v_unweighted", graph="chung_lu", weights="none", n=200003, length=40),
        # Weighted DeepWalk corpus on the benchmark's graph.
        _case("deepwalk_large", scale=22, weights="zipf", algo="deepwalk", n=524288),
        # DeepWalk without weights: every neighbour equally likely.
        _case("deepwalk_unweighted", scale=21, weights="none", algo="deepwalk", n=1000003),
        # Personalised PageRank by Monte Carlo: all walks from one hub.
        _case("ppr_hub", scale=22, weights="zipf", algo="ppr", n=1048576, starts="hub"),
        # MetaPath over edge labels, many walks of moderate length.
        _case("metapath_large", graph="chung_lu", scale=22, weights="none", labels=True,
              algo="metapath", n=2097152, length=20),
        # The paper's direct reservoir sampler as the pick rule.
        _case("deepwalk_dprs", entry="dprs", algo="deepwalk", n=50021, length=20),
        # Rows wanted in host memory (a trainer on the CPU side reads them).
        _case("deepwalk_host", entry="host", algo="deepwalk", n=100003),
        # A burst of requests of mixed algorithms and sizes at the server.
        _case("served_mix", entry="served", labels=True, algo="mixed", n=64, length=80),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    use = rng.choice(["small", "batch", "large", "large", "dprs", "host", "served"])
    if use == "served":
        return _case(None, entry="served", scale=rng.randint(16, 20), labels=True, algo="mixed",
                     weights="uniform", n=_log(rng, 4, 64), length=rng.randint(20, 80))
    algo = rng.choice(["node2vec", "node2vec", "deepwalk", "metapath", "ppr"])
    n = {"small": (1, 64), "batch": (64, 30000), "large": (30000, 524288),
         "dprs": (1000, 50000), "host": (10000, 100003)}[use]
    scale = rng.randint(18, 21) if use == "large" else rng.randint(12, 20)
    starts = "hub" if algo == "ppr" and rng.random() < 0.5 else "uniform"
    return _case(None, entry=use if use in ("dprs", "host") else "walk",
                 graph=rng.choice(["rmat", "rmat", "chung_lu"]), scale=scale,
                 edge_factor=rng.randint(6, 16), algo=algo, labels=algo == "metapath",
                 weights=rng.choice(["none", "uniform", "zipf"]), n=_log(rng, *n),
                 length=rng.randint(5, 20) if use == "dprs" else rng.randint(10, 80),
                 starts=starts)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _endpoints(case, gen):
    n = 1 << case["scale"]
    m = n * case["edge_factor"]
    if case["graph"] == "chung_lu":
        # Edge endpoints with expected degrees proportional to (i + 4)^(-1/1.1).
        c, i0 = 1 - 1 / 1.1, 4.0
        lo, hi = i0 ** c, (n + i0) ** c

        def ends():
            u = torch.rand(m, generator=gen, device="cuda", dtype=torch.float64)
            return ((lo + u * (hi - lo)) ** (1 / c) - i0).long().clamp_(0, n - 1)
        return n, ends(), ends()
    a = torch.zeros(m, dtype=torch.int64, device="cuda")
    b = torch.zeros_like(a)
    for _ in range(case["scale"]):
        u = torch.rand(m, generator=gen, device="cuda")
        right = ((u >= 0.57) & (u < 0.76)) | (u >= 0.95)
        down = u >= 0.76
        a.mul_(2).add_(down)
        b.mul_(2).add_(right)
    return n, a, b


def _mix(x):
    """A 32-bit hash of int64 values (as int64 in [0, 2^32))."""
    for mul in (0x2545F4914F6CDD1D, 0x5851F42D4C957F2D):
        x = x * mul
        x = x ^ ((x >> 32) & 0xFFFFFFFF)
    return x & 0xFFFFFFFF


def _graph(case, seed):
    """Host CSR arrays (offsets, adj, weights, labels) of the case's graph."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    salt = (seed * 0x9E3779B97F4A7C15 + 1) & (MASK >> 2)
    n, a, b = _endpoints(case, gen)
    ids = torch.randperm(n, generator=gen, device="cuda")
    a, b = ids[a], ids[b]
    keep = a != b
    a, b = a[keep], b[keep]
    keys = torch.cat([a * n + b, b * n + a])
    del a, b, keep, ids
    keys = torch.unique_consecutive(keys.sort()[0])
    src, dst = keys // n, keys % n
    edge = torch.minimum(src, dst) * n + torch.maximum(src, dst)
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.bincount(src, minlength=n).cumsum(0)
    weights = labels = None
    if case["weights"] == "uniform":
        weights = (1 + _mix(edge ^ salt) % 255).int().cpu().numpy().view(np.uint32)
    elif case["weights"] == "zipf":
        k = torch.arange(1, 65536, dtype=torch.float64, device="cuda")
        cum = (k ** -1.2).cumsum(0) / ZETA_1_2
        u = _mix(edge ^ salt).double() / 2.0 ** 32
        weights = (1 + torch.searchsorted(cum, u, right=True)).clamp_(max=65535)
        weights = weights.int().cpu().numpy().view(np.uint32)
    if case["labels"]:
        labels = (_mix((edge ^ salt) + 77) % 5).to(torch.uint8).cpu().numpy()
    return (off.cpu().numpy().view(np.uint64), dst.int().cpu().numpy().view(np.uint32),
            weights, labels)


def _starts(case, seed, off):
    n = off.shape[0] - 1
    if case["starts"] == "hub":
        return np.full(case["n"], int(np.argmax(np.diff(off))), dtype=np.uint32)
    return np.random.default_rng(seed + 1).integers(0, n, case["n"], dtype=np.uint32)


def _params(algo):
    if algo == "node2vec":
        return fw.make_params(FACTORS)
    if algo == "metapath":
        return fw.make_params(schema=SCHEMA)
    if algo == "ppr":
        return fw.make_params(stop=STOP)
    return None


def _requests(case, seed, n_vertices):
    """A burst of requests: sizes log-uniform in [1, 8192], lengths up to the
    case's, DeepWalk, node2vec and MetaPath in turn (the same sizes and lengths
    whatever the seed)."""
    sizes = np.random.default_rng(case["n"])
    rng = np.random.default_rng(seed + 2)
    out = []
    for i in range(case["n"]):
        algo = ("deepwalk", "node2vec", "metapath")[i % 3]
        k = int(math.exp(sizes.uniform(0, math.log(8192))))
        length = int(sizes.integers(max(1, case["length"] // 4), case["length"] + 1))
        starts = rng.integers(0, n_vertices, k, dtype=np.uint32)
        out.append((algo, _params(algo), starts, length, int(rng.integers(1 << 32))))
    return out


def prepare(case, seed):
    off, adj, weights, labels = _graph(case, seed)
    state = dict(case=case, seed=(seed + 42) & MASK, prm=_params(case["algo"]),
                 graph=fw.Graph.upload(off, adj, weights, labels))
    if case["entry"] == "served":
        state["requests"] = _requests(case, seed, off.shape[0] - 1)
        state["server"] = fw.Server(state["graph"], mem_budget_bytes=256 << 20)
        return state
    starts = _starts(case, seed, off)
    state["starts"] = (starts if case["entry"] == "host"
                       else torch.from_numpy(starts.view(np.int32)).cuda())
    torch.cuda.empty_cache()
    return state


def run(state):
    case = state["case"]
    if case["entry"] == "served":
        srv = state["server"]
        tickets = [srv.submit(*r) for r in state["requests"]]
        return [srv.wait(t)[0] for t in tickets]
    args = (state["graph"], case["algo"], state["prm"], state["starts"], case["length"],
            state["seed"])
    if case["entry"] == "host":
        return fw.walk_host(*args)[0]
    if case["entry"] == "dprs":
        return fw.walk(*args, mode="plain", sampler="dprs")
    return fw.walk(*args)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _mean_degree(case):
    """About how many neighbours a hop has: the degree of a vertex met with
    chance proportional to its degree, less what repeated draws of an edge,
    merged, take off the hubs (about half of it on these graphs).  Where all
    walks start at one hub its row, which they share, is left out."""
    n = float(1 << case["scale"])
    m2 = 2 * n * case["edge_factor"]
    if case["graph"] == "chung_lu":
        c, i0 = 1 - 1 / 1.1, 4.0
        z = (n + i0) ** c - i0 ** c
        p2 = (c / z) ** 2 * (i0 ** (2 * c - 1) - (n + i0) ** (2 * c - 1)) / (1 - 2 * c)
        return 0.3 * m2 * p2 + 1
    return 0.57 * m2 * (0.76 ** 2 + 0.24 ** 2) ** case["scale"] + 1


def work(case):
    """What a walk that keeps no per-vertex state cannot do without: per hop
    two row bounds, the row's entries that the algorithm has to see (every
    weight, every label; for node2vec also the ids of the shorter of the two
    rows and as many of the longer one's), the id picked and the entry
    written.  Operations: one add per entry seen, one multiply more for
    node2vec.  Rows met again count again: the graphs are larger than the
    caches, save the smallest, whose hubs' rows come from there."""
    n, length, algo, d = case["n"], case["length"], case["algo"], _mean_degree(case)
    hops = float(n * length)
    if case["graph"] == "rmat" and case["starts"] == "uniform":
        hops *= 0.6  # the other starts are isolated vertices
    if algo == "mixed":
        hops, algo = hops * 700 * 0.62, "node2vec"
    elif algo == "metapath":
        hops *= 0.53  # a label that no neighbour carries ends the walk
    elif algo == "ppr":
        hops *= min(1.0, (STOP[1] / STOP[0] - 1) / length)
    seen = float(d if case["weights"] != "none" or algo == "metapath" else 0)
    size = (1 if algo == "metapath" else 0) + (4 if case["weights"] != "none" else 0)
    extra = 2 * d * (0.18 if case["graph"] == "rmat" else 0.035) if algo == "node2vec" else 0.0
    rows = 4.0 * (hops if case["entry"] == "served" else n * (length + 1))
    return {"bytes": hops * (size * seen + 4 * extra + 16 + 4) + rows,
            "flops": hops * ((seen + extra) * (2 if algo == "node2vec" else 1) + 1)}


# ---------------------------------------------------------------------------
# The rows themselves, from the definition
# ---------------------------------------------------------------------------
def _philox(c0, c1, seed):
    """Words 0 and 1 of Philox4x64-10 (Salmon et al., SC 2011) at counter
    (c0, c1, 0, 0), key (seed, 0)."""
    c, k = [c0, c1, 0, 0], [seed & MASK, 0]
    for _ in range(10):
        p0, p1 = 0xD2E7470EE14C6C93 * c[0], 0xCA5A826395121157 * c[2]
        c = [(p1 >> 64) ^ c[1] ^ k[0], p1 & MASK, (p0 >> 64) ^ c[3] ^ k[1], p0 & MASK]
        k = [(k[0] + 0x9E3779B97F4A7C15) & MASK, (k[1] + 0xBB67AE8584CAA73B) & MASK]
    return c[0], c[1]


def _walk_rows(case, off, adj, weights, labels, starts, seed):
    """Every hop by its definition: all transition weights of the row, their
    prefix sums, one draw, the first prefix above it."""
    algo, length = case["algo"], case["length"]
    rows = np.full((len(starts), length + 1), 0xFFFFFFFF, dtype=np.uint32)
    for q, s in enumerate(starts):
        cur, prev = int(s), None
        rows[q, 0] = cur
        for t in range(length):
            u0, u1 = _philox(q, t, seed)
            if algo == "ppr" and (u1 * STOP[1]) >> 64 < STOP[0]:
                break
            b, e = int(off[cur]), int(off[cur + 1])
            ids = adj[b:e]
            w = np.ones(e - b, np.uint64) if weights is None else weights[b:e].astype(np.uint64)
            if algo == "node2vec" and prev is not None:
                near = np.isin(ids, adj[int(off[prev]):int(off[prev + 1])])
                f = np.where(ids == prev, FACTORS[0], np.where(near, FACTORS[1], FACTORS[2]))
                w = w * f.astype(np.uint64)
            elif algo == "metapath":
                w = w * (labels[b:e] == SCHEMA[t % len(SCHEMA)])
            prefix = np.cumsum(w, dtype=np.uint64)
            total = int(prefix[-1]) if e > b else 0
            if total == 0:
                break
            r = (u0 * total) >> 64
            prev, cur = cur, int(ids[np.searchsorted(prefix, np.uint64(r), side="right")])
            rows[q, t + 1] = cur
    return rows


def exact(case, seed):
    hops = case["n"] * min(case["length"], 5 if case["algo"] == "ppr" else 80)
    if case["entry"] != "walk" or hops * (200 + _mean_degree(case)) > 3e7:
        return None
    off, adj, weights, labels = _graph(case, seed)
    rows = _walk_rows(case, off, adj, weights, labels, _starts(case, seed, off), (seed + 42) & MASK)
    return torch.from_numpy(rows.view(np.int32))
