"""The persistent walker on few queries and on crowded caches of hub totals,
against the oracle bit for bit.

Launches of few queries take a workgroup per query unless the caller passes an
fw_tune, so every case here passes one.  Hub rows up to the longest class,
found in the cache with 64 and with 16 totals and descended from there; more
hub rows than the ways of their buckets hold, in both regions, with small and
with full workgroups, so that rows are replaced while other wavefronts read
them; node2vec's switch to searches of N(prev)."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip
from helpers import tiny6
from test_gpu_parity import (_BIG_STAR_ALGOS, _big_star, _labelled_hub, _ratio_boundary, _star,
                             _two_hubs)

pytestmark = pytest.mark.gpu

PERSISTENT = dict(wgs_per_cu=8)


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    return torch, fw


def _check(env, g, algo, factors, schema, stop, starts, length, seed, exp=None, **tune):
    torch, fw = env
    G = fw.Graph.of(g)
    got = gpu_walk(torch, fw, G, algo, fw.make_params(factors, schema, stop), starts, length, seed,
                   "persistent", tune=fw.make_tune(**(tune or PERSISTENT)))
    if exp is None:
        ids = np.arange(len(starts), dtype=np.uint64)
        exp = oracle.walk_ids_threaded(g, algo, oracle.params(*factors, schema=schema, stop=stop),
                                       starts, ids, length, seed, 16)
    assert_rows_equal(got, exp, f"{algo} n={len(starts)} L={length} {tune}")
    G.free()
    return exp


ALGOS = [("deepwalk", (1, 1, 1), (), (0, 1)), ("node2vec", (2, 3, 5), (), (0, 1)),
         ("metapath", (1, 1, 1), (0, 1, 2), (0, 1)), ("ppr", (1, 1, 1), (), (1, 9))]


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("length", [1, 5, 70])
def test_tiny6_node2vec(env, weighted, length):
    g, _ = tiny6(weighted=weighted)
    starts = np.tile(np.arange(6, dtype=np.uint32), 40)
    for f in ((1, 2, 4), (4, 2, 1)):
        _check(env, g, "node2vec", f, (), (0, 1), starts, length, 99)


@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
@pytest.mark.parametrize("d", [65, 4097, 70_000, 300_001])
def test_stars(env, algo, factors, schema, stop, d):
    g = _star(d, d)
    starts = np.concatenate([np.zeros(64, np.uint32), np.arange(1, 41, dtype=np.uint32)])
    _check(env, g, algo, factors, schema, stop, starts, 9, 1234)


@pytest.mark.parametrize("d,lead", [(16385, 2), (114691, 3), (131073, 1), (300001, 2)])
def test_metapath_hub_rows(env, d, lead):
    g = _labelled_hub(d, lead)
    starts = np.concatenate([np.ones(96, np.uint32), np.arange(2, 34, dtype=np.uint32)])
    for schema in [(1,), (2, 0)]:
        _check(env, g, "metapath", (1, 1, 1), schema, (0, 1), starts, 6, 4242 + d)


@pytest.mark.parametrize("algo,factors,schema,stop", _BIG_STAR_ALGOS)
@pytest.mark.parametrize("d", [1_048_577, 2_840_149])
def test_longest_rows(env, algo, factors, schema, stop, d):
    """Each workgroup visits the hub about a dozen times: the first visit leaves
    its totals, the others start from them.  256 cells leave node2vec room for
    the region of 64 totals; its default of 1,024 for 16 totals only, whose
    groups are four times as long."""
    g = _big_star(d, d)
    starts = np.concatenate([np.zeros(24, np.uint32), np.arange(1, 25, dtype=np.uint32),
                             np.array([d, d - 1, d // 2], np.uint32)])
    exp = _check(env, g, algo, factors, schema, stop, starts, 6, 4321)
    if algo == "node2vec":
        _check(env, g, algo, factors, schema, stop, starts, 6, 4321, exp, wgs_per_cu=8,
               hash_cells=256)


@pytest.mark.parametrize("d", [100, 5000, 40000])
def test_hub_to_hub(env, d):
    g = _two_hubs(d)
    starts = np.array([0, 1] * 64 + list(range(2, min(200, d + 2))), dtype=np.uint32)
    for f in ((4, 2, 1), (1, 2, 4)):
        _check(env, g, "node2vec", f, (), (0, 1), starts, 12, 5)


@pytest.mark.parametrize("cells", [512, 2048])
@pytest.mark.parametrize("pd", [640, 641])
def test_search_ratio(env, cells, pd):
    """N(prev) at 32x N(cur) (merge with 512 cells, hash set with 2,048) and one
    entry past it (binary search of the row)."""
    g = _ratio_boundary(20, pd)
    starts = np.tile(np.arange(1, 65, dtype=np.uint32), 4)
    for f in [(4, 2, 1), (1, 2, 4)]:
        _check(env, g, "node2vec", f, (), (0, 1), starts, 12, 2024, hash_cells=cells,
               sparse_ratio=0xFFFFFFFF)


# ---------------------------------------------------------------------------
# Crowded caches.  Geometry and hash as in fw_hub_cache.h and launch_any; only
# how crowded the buckets get hangs on them, not what is right.
# ---------------------------------------------------------------------------
WAYS = 4


def _buckets(algo, wgs, block, cells):
    budget = 160 * 1024 * (block // 256) // max(wgs, 8) // 1280 * 1280
    words = (budget - (cells * 4 * (block // 64) if algo == "node2vec" else 0)) // 4
    first = words // 4 // (3 * WAYS + WAYS * 64)
    return first, (words - first * (3 * WAYS + WAYS * 64)) // (3 * WAYS + WAYS * 16)


def _bucket_of(v, n):
    return (v.astype(np.uint64) * np.uint64(0x9E3779B1) % np.uint64(2**32) * np.uint64(n)) >> 32


def _crowd(first, few, n_long, n_short, seed):
    """Hubs whose totals all belong to one bucket of the second region and, the
    n_long longer ones, to one of the first; all degrees distinct."""
    nv = 40_000
    ids = np.arange(nv, dtype=np.uint32)
    fb, sb = _bucket_of(ids, first), _bucket_of(ids, few)
    rng = np.random.default_rng(seed)
    pool = ids[sb == sb[17]]
    both = pool[_bucket_of(pool, first) == fb[17]]
    long_ids = rng.permutation(both)[:n_long]
    short_ids = rng.permutation(np.setdiff1d(pool, long_ids))[:n_short]
    assert len(long_ids) == n_long > WAYS and len(short_ids) == n_short > WAYS
    hubs = np.concatenate([long_ids, short_ids])
    deg = np.concatenate([32_768 + 150 * np.arange(n_long), 2048 + 130 * np.arange(n_short)])
    leaves = np.setdiff1d(ids, hubs)
    src, dst, w = [], [], []
    for k in rng.permutation(len(hubs)):  # so that no order of visits follows the degree
        src.append(np.full(deg[k], hubs[k], np.int64))
        dst.append(rng.choice(leaves, deg[k], replace=False).astype(np.int64))
        # A leaf's edge to a short hub weighs more: both kinds are visited.
        w.append(rng.integers(1, 100, deg[k]) * (1 if k < n_long else 12))
    s, t, w = np.concatenate(src), np.concatenate(dst), np.concatenate(w).astype(np.uint32)
    lab = rng.integers(0, 3, s.size).astype(np.uint8)
    a, b = np.concatenate([s, t]), np.concatenate([t, s])
    order = np.lexsort((b, a))
    off = np.zeros(nv + 1, np.uint64)
    off[1:] = np.cumsum(np.bincount(a, minlength=nv))
    return SimpleNamespace(offsets=off, adj=b[order].astype(np.uint32),
                           weights=np.concatenate([w, w])[order],
                           labels=np.concatenate([lab, lab])[order], n_vertices=nv,
                           n_edges=2 * s.size), leaves


@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
@pytest.mark.parametrize("wgs,block,n", [(1, 256, 3000), (4, 1024, 4096)])
def test_crowded_buckets(env, algo, factors, schema, stop, wgs, block, n):
    """Every workgroup's walks meet 8 long and 24 short hubs, all in one bucket
    of their region: four stay, the others replace shorter ones, fall back to
    the second region or are streamed."""
    first, few = _buckets(algo, wgs, block, 256)
    assert first >= 1 and few >= 4
    g, leaves = _crowd(first, few, 8, 24, seed=wgs)
    starts = leaves[(np.arange(n, dtype=np.uint64) * 7919 % len(leaves)).astype(np.int64)]
    _check(env, g, algo, factors, schema, (0, 1) if algo == "ppr" else stop, starts, 40, 55,
           wgs_per_cu=wgs, hash_cells=256)
    if algo == "metapath":  # one label: its keys share the buckets too
        _check(env, g, algo, factors, (0,), stop, starts, 40, 56, wgs_per_cu=wgs, hash_cells=256)
