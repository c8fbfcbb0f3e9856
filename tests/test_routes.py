"""Which kernel a walk launches (CPU, over the host-memory runtime): by query
count, weights, the longest row and whether the caller passes an fw_tune."""
import json

import pytest

from host_hip import host_hip  # noqa: F401  (fixture)

ALGOS = ["deepwalk", "node2vec", "metapath", "ppr"]
# Queries per CU (of 256) up to which an untuned launch takes a workgroup per
# query: on graphs with a row past 8,192 entries, without one, without weights.
LONG = {"deepwalk": 12, "node2vec": 12, "metapath": 4, "ppr": 12}
SHORT = {"deepwalk": 0, "node2vec": 3, "metapath": 0, "ppr": 0}


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("hub", [8192, 8193])
def test_kernel_of_a_launch(host_hip, hub, weighted):  # noqa: F811
    got = json.loads(host_hip(f"""
import json
prm = {{"deepwalk": None, "node2vec": fw.make_params((1, 2, 4)),
       "metapath": fw.make_params(schema=(0, 1)), "ppr": fw.make_params(stop=(1, 5))}}
g = ring(hub={hub} - 1, **({{}} if {weighted} else dict(weights=None)))
assert g.info()["max_degree"] == {hub}
st = np.zeros(4000, np.uint32)
rows = np.zeros((4000, 3), np.uint32)
out = {{}}
for a in {ALGOS!r}:
    for n in (1, 768, 769, 1024, 1025, 3072, 3073):
        for tune in (None, fw.make_tune(wgs_per_cu=8)):
            launches()
            assert fw.walk_ptr(g, a, prm[a], st.ctypes.data, n, 2, 1, rows.ctypes.data,
                               mode="persistent", tune=tune) == 0
            (l,) = launches()
            name = l.name.decode()
            (k,) = [k for k in ("team", "uniform", "persistent") if "k_walk_" + k in name]
            out[f"{{a}} {{n}} {{'tuned' if tune else 'default'}}"] = k
print(json.dumps(out))
"""))
    for key, kernel in got.items():
        algo, n, how = key.split()
        unit = not weighted and algo in ("deepwalk", "ppr")
        per_cu = 0 if unit else (LONG if hub > 8192 else SHORT)[algo]
        if how == "default" and int(n) <= 256 * per_cu:
            assert kernel == "team", key
        else:
            assert kernel == ("uniform" if unit else "persistent"), key
