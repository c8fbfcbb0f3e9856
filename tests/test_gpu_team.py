"""Small launches (a workgroup per query) against the oracle, bit for bit:
query counts around the changes of the workgroup's size, rows around one chunk
of 256 entries, one group per chunk and the longest rows (groups of several
chunks, descended again), N(prev) around the leader's and the workgroup's hash
sets and past them, walks past 64 hops, early ends."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip
from helpers import csr_from_edges

pytestmark = pytest.mark.gpu

ALGOS = [("deepwalk", (1, 1, 1), (), (0, 1)), ("ppr", (1, 1, 1), (), (1, 9)),
         ("metapath", (1, 1, 1), (0, 1, 2), (0, 1)), ("node2vec", (2, 3, 5), (), (0, 1))]


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    return torch, fw


def _check(env, g, algo, factors, schema, stop, starts, length, seed=8, **tune):
    """tune: run the persistent form so configured instead."""
    torch, fw = env
    G = fw.Graph.of(g)
    got = gpu_walk(torch, fw, G, algo, fw.make_params(factors, schema, stop), starts, length, seed,
                   "auto", qid_base=3, tune=fw.make_tune(**tune) if tune else None)
    exp = oracle.walk(g, algo, oracle.params(*factors, schema=schema, stop=stop), starts, length,
                      seed, qid_base=3)
    assert_rows_equal(got, exp, f"{algo} n={len(starts)} L={length}")
    G.free()


def _clique_star(d, k, seed, weighted):
    """Hub 0 joined to vertices 1..d, and k of those (odd ids first) joined to
    hub d + 1 too: node2vec hops between two long rows that share entries."""
    rng = np.random.default_rng(seed)
    e = [(0, i + 1, int(rng.integers(1, 2**16)), int(rng.integers(0, 3))) for i in range(d)]
    shared = np.concatenate([np.arange(1, d + 1, 2), np.arange(2, d + 1, 2)])[:k]
    e += [(d + 1, int(v), int(rng.integers(1, 2**16)), int(rng.integers(0, 3))) for v in shared]
    e += [(0, d + 1, 500 * d, 1)]  # the hubs meet often
    return csr_from_edges(d + 2, e, weights=weighted)


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
@pytest.mark.parametrize("d,k", [(1, 1), (255, 3), (256, 256), (257, 200), (1027, 600),
                                 (17_000, 9_000), (40_000, 20_000)])
def test_row_lengths(env, algo, factors, schema, stop, d, k, weighted):
    g = _clique_star(d, k, d, weighted)
    starts = np.concatenate([[0, d + 1, 0, d + 1], 1 + np.arange(min(d, 20))]).astype(np.uint32)
    _check(env, g, algo, factors, schema, stop, starts, 7)
    _check(env, g, algo, factors, schema, stop, starts, 7, wgs_per_cu=8)


@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
def test_longest_rows(env, algo, factors, schema, stop):
    """300,001 entries: groups of two chunks with sixteen wavefronts, of three
    with eight, of ten with two."""
    g = _clique_star(300_001, 5_000, 9, True)
    for n in (40, 600, 1100):
        starts = np.arange(n, dtype=np.uint32) % 5 * 17
        _check(env, g, algo, factors, schema, stop, starts, 3)


@pytest.mark.parametrize("algo,factors,schema,stop", ALGOS)
@pytest.mark.parametrize("n,length", [(1, 200), (3, 0), (5, 1), (255, 63), (256, 64), (257, 65),
                                      (512, 20), (768, 20), (769, 20)])
def test_counts_and_lengths(env, algo, factors, schema, stop, n, length):
    g = synth.rmat(13, 6, seed=71)  # isolated vertices and hubs
    g.weights = synth.weights_zipf(g, 1.2, 65535, 72)
    g.labels = synth.labels_uniform(g, 3, 73)
    starts = (np.arange(n, dtype=np.uint64) * 2654435761 % g.n_vertices).astype(np.uint32)
    _check(env, g, algo, factors, schema, stop, starts, length)


def test_invalid_start(env):
    torch, fw = env
    g = synth.rmat(10, 6, seed=74)
    g.weights = synth.weights_uniform(g, 1, 255, 75)
    G = fw.Graph.of(g)
    st = torch.tensor([1, g.n_vertices, 2], dtype=torch.int32, device="cuda")
    out = torch.empty((3, 6), dtype=torch.int32, device="cuda")
    with pytest.raises(fw.FWError):
        fw.walk(G, "deepwalk", None, st, 5, 1, out=out)
    exp = oracle.walk(g, "deepwalk", oracle.params(), np.array([1, 0, 2], np.uint32), 5, 1)
    assert_rows_equal(out.cpu().numpy().view(np.uint32)[[0, 2]], exp[[0, 2]], "valid starts")
    G.free()
