"""DPRS picked from the last chunk backwards, against the oracle bit for bit:
rows around one and several 256-entry chunks, totals around 32 bits, rows whose
last chunks weigh nothing, more queries than wavefronts."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip
from helpers import csr_from_edges

pytestmark = pytest.mark.gpu

ALGOS = [("deepwalk", (), (0, 1)), ("ppr", (), (1, 5)), ("metapath", (0, 1, 2), (0, 1))]


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    return torch, fw


def _check(env, g, algo, sch, stop, starts, length, weighted=True):
    torch, fw = env
    if not weighted:
        g.weights = None
    G = fw.Graph.of(g)
    got = gpu_walk(torch, fw, G, algo, fw.make_params((1, 1, 1), sch, stop), starts, length, 77,
                   "plain", qid_base=9, sampler="dprs")
    exp = oracle.walk(g, algo, oracle.params(1, 1, 1, schema=sch, stop=stop), starts, length, 77,
                      qid_base=9, sampler="dprs")
    assert_rows_equal(got, exp, f"{algo} n={len(starts)}")
    G.free()


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("algo,sch,stop", ALGOS)
@pytest.mark.parametrize("d,heavy,zeros", [(1, 9, 0), (4, 9, 0), (255, 9, 0), (256, 9, 0),
                                           (257, 9, 0), (1025, 9, 700), (513, 2**23, 0),
                                           (600, 2**32 - 1, 300), (1024, 2**22, 0)])
def test_rows(env, algo, sch, stop, d, heavy, zeros, weighted):
    rng = np.random.default_rng(d + zeros)
    e = []
    for i in range(d):
        w = 0 if i >= d - zeros else int(rng.integers(1, heavy, endpoint=True))
        e.append((0, i + 1, w, int(rng.integers(0, 3))))
    g = csr_from_edges(d + 1, e)
    starts = np.concatenate([np.zeros(60, np.uint32), np.arange(min(d, 9) + 1, dtype=np.uint32)])
    _check(env, g, algo, sch, stop, starts, 4, weighted)


@pytest.mark.parametrize("algo,sch,stop", ALGOS)
def test_more_queries_than_wavefronts(env, algo, sch, stop):
    g = synth.rmat(12, 4, seed=5)
    g.weights = synth.weights_uniform(g, 0, 255, 6)
    g.labels = synth.labels_uniform(g, 3, 7)
    starts = (np.arange(30_011, dtype=np.uint64) * 40503 % g.n_vertices).astype(np.uint32)
    _check(env, g, algo, sch, stop, starts, 5)
