"""fw_walk_host calls of growing and shrinking results on one graph: the pinned
slots it keeps are replaced by larger ones or used in part, in one batch and in
several, against fw_walk."""
import numpy as np
import pytest

import synth
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip

pytestmark = pytest.mark.gpu


def test_sizes_in_turn():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    g = synth.rmat(14, 8, seed=21)
    g.weights = synth.weights_uniform(g, 1, 255, 22)
    G = fw.Graph.of(g)
    # Rows of 16 entries: 64 bytes to 19 MB; a length of 0 (rows of one entry)
    # takes as many bytes in as out.
    for n, cap, length in ((1, 0, 15), (3000, 0, 15), (20_000, 0, 15), (1, 0, 15), (300_000, 0, 15),
                           (300_001, 150_000, 15), (17, 5, 15), (100_003, 20_000, 15),
                           (900_000, 0, 0), (900_000, 300_001, 0), (65_537, 0, 15)):
        starts = (np.arange(n, dtype=np.uint64) * 2654435761 % g.n_vertices).astype(np.uint32)
        rows, _, nb = fw.walk_host(G, "deepwalk", None, starts, length, 9, max_batch_queries=cap)
        assert nb == (-(-n // cap) if cap else 1)
        assert_rows_equal(rows, gpu_walk(torch, fw, G, "deepwalk", None, starts, length, 9, "auto"),
                          f"n={n} cap={cap} L={length}")
    G.free()
