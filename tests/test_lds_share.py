"""LDS that launches of the persistent walker ask for (CPU, over the
host-memory runtime).  A launch that is given fewer workgroups per CU than the
eight of 256 threads the kernel is built for shares the CU with other launches:
it may take an eighth of the CU's LDS per workgroup, so that what runs beside
it finds room."""
import json

import pytest

from host_hip import host_hip  # noqa: F401  (fixture)

CUS, CU_LDS, GRAIN = 256, 160 * 1024, 1280
ALGOS = ["deepwalk", "node2vec", "metapath", "ppr"]

COMMON = """
import json
prm = {"deepwalk": None, "node2vec": fw.make_params((1, 2, 4)),
       "metapath": fw.make_params(schema=(0, 1)), "ppr": fw.make_params(stop=(1, 5))}
out = {}
def cu_lds(l):
    per_cu = -(-l.grid // 256)
    return per_cu * (-(-l.lds // 1280) * 1280)
"""


@pytest.mark.parametrize("inflight", [2, 3, 4, 7])
def test_bulk_and_express_fit_a_cu(host_hip, inflight):  # noqa: F811
    """Every bulk stream's launch and an express launch, all as large as they
    get, are resident on a CU together."""
    got = json.loads(host_hip(COMMON + f"""
g = ring()
srv = fw.Server(g, mem_budget_bytes=64 << 20, max_inflight={inflight}, express_max_queries=20000)
for a in {ALGOS!r}:
    for what, n in (("bulk", 120000), ("express", 20000)):
        launches()
        srv.wait(srv.submit(a, prm[a], np.zeros(n, np.uint32), 4, 1))
        (l,) = launches()
        assert b"k_walk_persistent" in l.name
        out.setdefault(a, {{}})[what] = (cu_lds(l), l.grid * l.block // 256)
srv.close()
print(json.dumps(out))
"""))
    bulk_wgs = max(1, 6 // (inflight - 1))
    for bulk in ALGOS:
        for express in ALGOS:
            b, e = got[bulk]["bulk"], got[express]["express"]
            assert b[1] == bulk_wgs * CUS and e[1] == 2 * CUS
            assert (inflight - 1) * b[0] + e[0] <= CU_LDS, (bulk, express)


@pytest.mark.parametrize("wgs", [1, 2, 3, 4, 5, 6, 7, 8, 12, 16])
def test_configured_share(host_hip, wgs):  # noqa: F811
    """fw_tune.wgs_per_cu = k of 8: at most k eighths of the LDS, or what
    node2vec's regions take if that is more."""
    got = json.loads(host_hip(COMMON + f"""
g = ring()
st = np.zeros(400000, np.uint32)
rows = np.zeros((400000, 5), np.uint32)
for a in {ALGOS!r}:
    for cells in (64, 1024, 2048):
        launches()
        rc = fw.walk_ptr(g, a, prm[a], st.ctypes.data, st.size, 4, 1, rows.ctypes.data,
                         mode="persistent", tune=fw.make_tune(wgs_per_cu={wgs}, hash_cells=cells))
        assert rc == 0
        (l,) = launches()
        out[a + str(cells)] = (cu_lds(l), l.grid * l.block // 256)
print(json.dumps(out))
"""))
    for a in ALGOS:
        for cells in (64, 1024, 2048):
            lds, threads256 = got[a + str(cells)]
            assert threads256 == wgs * CUS
            share = CU_LDS * min(wgs, 8) // 8
            regions = wgs * -(-16 * cells // GRAIN) * GRAIN if a == "node2vec" else 0
            assert lds <= max(share, regions), (a, cells, lds)


def test_default_launch_uses_all_of_it(host_hip):  # noqa: F811
    """A launch that has the chip to itself: two workgroups of 1,024 threads
    per CU, each with the kept totals in what the regions leave of a half."""
    got = json.loads(host_hip(COMMON + """
g = ring(hub=9000)
st = np.zeros(400000, np.uint32)
rows = np.zeros((400000, 5), np.uint32)
for a in ("deepwalk", "node2vec"):
    launches()
    assert fw.walk_ptr(g, a, prm[a], st.ctypes.data, st.size, 4, 1, rows.ctypes.data) == 0
    (l,) = launches()
    out[a] = (cu_lds(l), l.grid, l.block)
print(json.dumps(out))
"""))
    for a, (lds, grid, block) in got.items():
        assert (grid, block) == (2 * CUS, 1024)
        assert CU_LDS * 0.97 < lds <= CU_LDS, a


@pytest.mark.parametrize("hub", [0, 9000])
def test_launches_of_few_wavefronts(host_hip, hub):  # noqa: F811
    """A launch that leaves wavefront slots free leaves as large a part of the
    LDS for the launches of other streams."""
    got = json.loads(host_hip(COMMON + f"""
g = ring(hub={hub})
st = np.zeros(8000, np.uint32)
rows = np.zeros((8000, 5), np.uint32)
for a in {ALGOS!r}:
    for n in (769, 1024, 1500, 3073, 3500, 4096, 5000, 8000):
        launches()
        assert fw.walk_ptr(g, a, prm[a], st.ctypes.data, n, 4, 1, rows.ctypes.data) == 0
        (l,) = launches()
        if b"k_walk_persistent" in l.name:
            out[f"{{a}} {{n}}"] = (cu_lds(l), -(-l.grid // 256) * l.block // 256)
print(json.dumps(out))
"""))
    assert any(k.startswith("node2vec 4096") for k in got)
    for k, (lds, wgs) in got.items():
        assert lds <= CU_LDS * wgs // 8, k


def test_no_hub_totals_where_none_are_read(host_hip):  # noqa: F811
    """Only node2vec's regrouped totals of weighted rows read the hub totals:
    without weights, or without that pass, a launch takes its regions alone."""
    got = json.loads(host_hip(COMMON + """
st = np.zeros(400000, np.uint32)
rows = np.zeros((400000, 5), np.uint32)
for what, kw, tune in (("unweighted", dict(weights=None), dict(hash_cells=1024)),
                       ("unweighted small", dict(weights=None), dict(hash_cells=256)),
                       ("never", {}, dict(hash_cells=512, sparse_ratio=0xFFFFFFFF)),
                       ("weighted", {}, dict(hash_cells=512))):
    g = ring(hub=9000, **kw)
    launches()
    assert fw.walk_ptr(g, "node2vec", prm["node2vec"], st.ctypes.data, st.size, 4, 1,
                       rows.ctypes.data, tune=fw.make_tune(**tune)) == 0
    (l,) = launches()
    out[what] = (l.lds, l.block // 64 * tune["hash_cells"] * 4)
print(json.dumps(out))
"""))
    for what, (lds, regions) in got.items():
        if what == "weighted":
            assert lds > regions
        else:
            assert lds == regions, what
