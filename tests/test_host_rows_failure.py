"""fw_walk_host when a later batch fails (CPU, over the host-memory runtime):
rows of batches that were not copied back keep what the caller had there."""
import json

import pytest

from host_hip import host_hip  # noqa: F401  (fixture)

N, BATCH, COLS = 60_000, 20_000, 16


@pytest.mark.parametrize("fail_at,copied", [(0, 0), (1, 0), (2, 1), (-1, 3)])
def test_rows_not_copied_are_left_alone(host_hip, fail_at, copied):  # noqa: F811
    got = json.loads(host_hip(f"""
import json
g = ring()
st = np.zeros({N}, np.uint32)
out = np.full(({N}, {COLS}), 0xA5A5A5A5, np.uint32)
o = fw.BatchOpts()
o.max_batch_queries = {BATCH}
launches()
hip.host_hip_fail_at({fail_at})
rc = fw.lib().fw_walk_host(g.handle, 0, None, st.ctypes.data, {N}, {COLS - 1}, 1,
                           out.ctypes.data, ctypes.byref(o))
kept = [bool((b == 0xA5A5A5A5).all()) for b in out.reshape(-1, {BATCH}, {COLS})]
gone = [bool((b == 0).all()) for b in out.reshape(-1, {BATCH}, {COLS})]
print(json.dumps(dict(rc=rc, kept=kept, gone=gone)))
"""))
    assert (got["rc"] == 0) == (fail_at < 0)
    # The runtime's kernels do not run: what is copied back is zeros.
    assert got["gone"] == [b < copied for b in range(3)]
    assert got["kept"] == [b >= copied for b in range(3)]
