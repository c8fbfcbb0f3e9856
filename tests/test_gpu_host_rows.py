"""Rows in host memory through the pinned slots: results around the size of a
slot and of the pieces, several batches whose copies alternate, calls at the
same time on one graph (the second makes its own staging), against fw_walk."""
import threading

import numpy as np
import pytest

import synth
from gpu_common import assert_rows_equal, gpu_walk, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = torch_or_skip()
    from paper_2404_08364_amd import flowwalk as fw
    g = synth.rmat(14, 8, seed=21)
    g.weights = synth.weights_uniform(g, 1, 255, 22)
    return torch, fw, g, fw.Graph.of(g)


# Rows of 16 entries: a slot holds 65,536 of them, a piece at least 4,096.
@pytest.mark.parametrize("n,cap", [(1, 0), (4095, 0), (4097, 0), (16_385, 0), (65_537, 0),
                                   (300_001, 0), (300_001, 70_000), (50_000, 16_384)])
def test_sizes(env, n, cap):
    torch, fw, g, G = env
    starts = (np.arange(n, dtype=np.uint64) * 2654435761 % g.n_vertices).astype(np.uint32)
    rows, B, nb = fw.walk_host(G, "deepwalk", None, starts, 15, 9, max_batch_queries=cap)
    assert B == (cap or n) and nb == -(-n // B)
    assert_rows_equal(rows, gpu_walk(torch, fw, G, "deepwalk", None, starts, 15, 9, "auto"),
                      f"n={n} cap={cap}")


def test_calls_at_the_same_time(env):
    torch, fw, g, G = env
    starts = np.arange(60_000, dtype=np.uint32) % g.n_vertices
    exp = [gpu_walk(torch, fw, G, "deepwalk", None, starts, 15, s, "auto") for s in range(3)]
    got = [None] * 3

    def call(s):
        for _ in range(3):
            got[s] = fw.walk_host(G, "deepwalk", None, starts, 15, s, max_batch_queries=25_000)[0]
    threads = [threading.Thread(target=call, args=(s,)) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in range(3):
        assert_rows_equal(got[s], exp[s], f"seed {s}")
