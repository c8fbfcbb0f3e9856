"""Plain node2vec against the oracle bit for bit, where N(prev) goes from the
LDS hash set to searches in global memory: rows of 512 entries and one to each
side, and rows 32 times as long as the current one and one to each side."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip
from helpers import csr_from_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("da,db", [(1, 1), (511, 300), (512, 300), (513, 300), (512, 16),
                                   (513, 16), (511, 16), (512, 15), (64, 2), (65, 2), (2000, 900)])
def test_membership(da, db, weighted):
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    # 0 and 1 are neighbours by a heavy edge and share half of the shorter row.
    rng = np.random.default_rng(1000 * da + db)
    e = [(0, 1, 5000, 0)]
    first = 2 + (da - 1) - min(da, db) // 2
    rows = [(0, range(2, 1 + da)), (1, range(max(2, first), max(2, first) + db - 1))]
    for hub, others in rows:
        for v in others:
            w = int(rng.integers(1, 10))
            e.append((hub, v, w, 0))
    n = 1 + max(max(x[0], x[1]) for x in e)
    g = csr_from_edges(n, e)
    assert g.offsets[1] - g.offsets[0] == da and g.offsets[2] - g.offsets[1] == db
    if not weighted:
        g.weights = None
    starts = np.concatenate([np.tile(np.array([0, 1], np.uint32), 150),
                             np.arange(min(n, 50), dtype=np.uint32)])
    G = fw.Graph.of(g)
    got = gpu_walk(torch, fw, G, "node2vec", fw.make_params((2, 4, 1)), starts, 12, 31, "plain")
    exp = oracle.walk(g, "node2vec", oracle.params(2, 4, 1), starts, 12, 31)
    assert_rows_equal(got, exp, f"da={da} db={db}")
    G.free()
