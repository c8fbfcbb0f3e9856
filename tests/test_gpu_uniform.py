"""Unweighted DeepWalk and PPR (a query per lane) against the oracle, bit for
bit: row lengths around the 16-entry store run, query counts around a
wavefront, a workgroup and past the grid (queries claimed from the counter),
early ends, invalid starts, and the served form."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    g = synth.rmat(13, 3, seed=77)  # about half of its vertices are isolated
    return torch, fw, g, fw.Graph.of(g)


CASES = [(n, length, 0) for n, length in [(1, 1), (15, 15), (63, 16), (64, 17), (65, 31), (257, 33),
                                          (300, 0), (4097, 14), (1000, 130)]]
CASES.append((140_003, 18, 2))  # 2 workgroups per CU: 131,072 lanes on 256 CUs


@pytest.mark.parametrize("algo,stop", [("deepwalk", (0, 1)), ("ppr", (1, 5)), ("ppr", (0, 1)),
                                       ("ppr", (1, 1))])
@pytest.mark.parametrize("n,length,wgs", CASES)
def test_rows(env, algo, stop, n, length, wgs):
    torch, fw, g, G = env
    starts = (np.arange(n, dtype=np.uint64) * 2654435761 % g.n_vertices).astype(np.uint32)
    prm = fw.make_params(stop=stop)
    got = gpu_walk(torch, fw, G, algo, prm, starts, length, 5, "persistent", qid_base=11,
                   tune=fw.make_tune(wgs_per_cu=wgs))
    exp = oracle.walk(g, algo, oracle.params(stop=stop), starts, length, 5, qid_base=11)
    assert_rows_equal(got, exp, f"{algo} n={n} L={length}")


def test_invalid_start_and_served(env):
    torch, fw, g, G = env
    bad = torch.tensor([1, g.n_vertices, 2], dtype=torch.int32, device="cuda")
    with pytest.raises(fw.FWError):
        fw.walk(G, "deepwalk", None, bad, 5, 1)
    srv = fw.Server(G, mem_budget_bytes=16 << 20)
    prm = fw.make_params(stop=(1, 4))
    reqs = [(("deepwalk", "ppr")[k % 2], np.arange(k, 7 * k + 1, 3, dtype=np.uint32), 10 + k, k)
            for k in range(1, 30)]
    tickets = [srv.submit(a, prm, s, length, seed) for a, s, length, seed in reqs]
    for (a, s, length, seed), t in zip(reqs, tickets):
        rows, st = srv.wait(t)
        exp = oracle.walk(g, a, oracle.params(stop=(1, 4)), s, length, seed)
        assert_rows_equal(rows, exp, f"served {a} seed {seed}")
        assert st["steps"] == int((exp[:, 1:] != 0xFFFFFFFF).sum())
    srv.close()
