"""How queries reach the persistent wavefronts: one, two and four to a
wavefront, and more than all of them hold (claims of several at a time), with
isolated and invalid starts among them, against the oracle bit for bit."""
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
    g = synth.rmat(13, 4, seed=78)  # many isolated vertices
    g.weights = synth.weights_uniform(g, 1, 255, 79)
    g.labels = synth.labels_uniform(g, 3, 80)
    return torch, fw, g, fw.Graph.of(g)


# One workgroup per CU: 1,024 wavefronts on 256 CUs.
@pytest.mark.parametrize("n", [1, 1023, 1025, 2049, 3073, 4095, 4097, 60_001])
@pytest.mark.parametrize("algo,factors,schema,stop", [
    ("deepwalk", (1, 1, 1), (), (0, 1)), ("ppr", (1, 1, 1), (), (1, 3)),
    ("metapath", (1, 1, 1), (0, 1, 2), (0, 1)), ("node2vec", (2, 3, 5), (), (0, 1))])
def test_rows(env, n, algo, factors, schema, stop):
    torch, fw, g, G = env
    starts = (np.arange(n, dtype=np.uint64) * 2654435761 % g.n_vertices).astype(np.uint32)
    got = gpu_walk(torch, fw, G, algo, fw.make_params(factors, schema, stop), starts, 19, 6,
                   "persistent", qid_base=5, tune=fw.make_tune(wgs_per_cu=1))
    exp = oracle.walk(g, algo, oracle.params(*factors, schema=schema, stop=stop), starts, 19, 6,
                      qid_base=5)
    assert_rows_equal(got, exp, f"{algo} n={n}")


def test_invalid_starts_do_not_stop_the_others(env):
    torch, fw, g, G = env
    starts = np.arange(9_000, dtype=np.uint32) % g.n_vertices
    starts[::7] = g.n_vertices
    st = torch.from_numpy(starts.view(np.int32)).cuda()
    out = torch.empty((9_000, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(fw.FWError):
        fw.walk(G, "deepwalk", None, st, 7, 3, out=out, tune=fw.make_tune(wgs_per_cu=1))
    good = np.ones(9_000, bool)
    good[::7] = False
    starts[::7] = 0
    exp = oracle.walk(g, "deepwalk", oracle.params(), starts, 7, 3)
    assert_rows_equal(out.cpu().numpy().view(np.uint32)[good], exp[good], "rows of valid starts")
