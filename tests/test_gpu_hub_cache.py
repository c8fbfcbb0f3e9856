"""Hub rows whose group totals the wavefronts of a workgroup share: more hubs
than the cache holds, rows around the smallest degree kept, totals past 32
bits, every algorithm that uses the totals, with full-size workgroups (the
launch fills the chip) and small ones, against the oracle bit for bit."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip

pytestmark = pytest.mark.gpu


def _hubs(n_hubs, n_leaves, lo, hi, max_w, seed):
    """n_hubs vertices joined to random leaves each, degrees in [lo, hi]."""
    rng = np.random.default_rng(seed)
    pairs = []
    for h in range(n_hubs):
        d = int(rng.integers(lo, hi + 1)) if h else 2048
        leaves = rng.choice(n_leaves, d, replace=False).astype(np.int64) + n_hubs
        pairs.append(np.stack([np.full(d, h, np.int64), leaves]))
    e = np.concatenate(pairs, axis=1)
    m = e.shape[1]
    w = rng.integers(1, max_w, m, endpoint=True).astype(np.uint32)
    lab = rng.integers(0, 3, m).astype(np.uint8)
    src, dst = np.concatenate([e[0], e[1]]), np.concatenate([e[1], e[0]])
    order = np.lexsort((dst, src))
    nv = n_hubs + n_leaves
    off = np.zeros(nv + 1, np.uint64)
    off[1:] = np.cumsum(np.bincount(src, minlength=nv))
    return SimpleNamespace(offsets=off, adj=dst[order].astype(np.uint32),
                           weights=np.concatenate([w, w])[order],
                           labels=np.concatenate([lab, lab])[order], n_vertices=nv,
                           n_edges=2 * m)


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    small = _hubs(500, 12_000, 1500, 5200, 1000, 3)  # 200+ row keys per workgroup and label
    wide = _hubs(40, 9_000, 2000, 8800, 2**32 - 1, 4)  # group totals past 32 bits among them
    bare = SimpleNamespace(**{**vars(small), "weights": None})
    long = _hubs(7, 60_000, 32_000, 45_000, 1000, 5)  # around the first region's smallest row
    return torch, fw, {"small": small, "wide": wide, "bare": bare, "long": long}


ALGOS = [("deepwalk", (1, 1, 1), (), (0, 1)), ("ppr", (1, 1, 1), (), (1, 20)),
         ("metapath", (1, 1, 1), (0, 1, 2), (0, 1)), ("node2vec", (2, 3, 5), (), (0, 1))]


@pytest.mark.parametrize("graph", ["small", "wide", "bare", "long"])
@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
@pytest.mark.parametrize("n,wgs", [(17_000, 4), (700, 0)])
def test_rows(env, graph, algo, factors, schema, stop, n, wgs):
    torch, fw, graphs = env
    g = graphs[graph]
    G = fw.Graph.of(g)
    starts = (np.arange(n, dtype=np.uint64) * 7919 % g.n_vertices).astype(np.uint32)
    got = gpu_walk(torch, fw, G, algo, fw.make_params(factors, schema, stop), starts, 6, 21,
                   "persistent", tune=fw.make_tune(wgs_per_cu=wgs))
    exp = oracle.walk(g, algo, oracle.params(*factors, schema=schema, stop=stop), starts, 6, 21)
    assert_rows_equal(got, exp, f"{algo} on {graph} n={n}")
    G.free()


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("algo,factors", [("deepwalk", (1, 1, 1)), ("node2vec", (2, 3, 5))])
def test_totals_around_32_bits(env, algo, factors, over):
    """Every weight at the largest value whose group totals are summed in 32
    bits (2^32 over the factor and d / 64 + 512 entries), and one above it."""
    torch, fw, _ = env
    d = 70_001
    limit = (2**32 - 1) // (max(factors) * (d // 64 + 512)) + over
    off = np.concatenate([[0, d], d + 1 + np.arange(d)]).astype(np.uint64)
    adj = np.concatenate([1 + np.arange(d), np.zeros(d)]).astype(np.uint32)
    g = SimpleNamespace(offsets=off, adj=adj, weights=np.full(2 * d, limit, np.uint32),
                        labels=None, n_vertices=d + 1, n_edges=2 * d)
    G = fw.Graph.of(g)
    starts = np.concatenate([np.zeros(40), np.arange(1, 60)]).astype(np.uint32)
    exp = oracle.walk(g, algo, oracle.params(*factors), starts, 5, 31)
    for tune in (None, fw.make_tune(wgs_per_cu=8)):
        got = gpu_walk(torch, fw, G, algo, fw.make_params(factors), starts, 5, 31, "persistent",
                       tune=tune)
        assert_rows_equal(got, exp, f"{algo} over={over}")
    G.free()
