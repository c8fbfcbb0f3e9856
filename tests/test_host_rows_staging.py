"""Pinned staging of fw_walk_host (CPU, over the host-memory runtime): a call
makes what its results need, later calls use it again, the graph gives it
back."""
import json

from host_hip import host_hip  # noqa: F401  (fixture)


def test_staging_follows_the_results(host_hip):  # noqa: F811
    got = json.loads(host_hip("""
import json
hip.host_hip_pinned.argtypes = [ctypes.c_void_p] * 3
def pinned():
    m, l, s = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_long()
    hip.host_hip_pinned(ctypes.byref(m), ctypes.byref(l), ctypes.byref(s))
    return m.value, l.value, s.value
g = ring()
out = []
base = pinned()
def call(n, cap=0):
    fw.walk_host(g, "deepwalk", None, np.zeros(n, np.uint32), 15, 1, max_batch_queries=cap)
    m, l, s = pinned()
    out.append((n, cap, m - base[0], l - base[1], s - base[2]))
# Rows of 64 bytes: 64 B, 640 KB, 1.3 MB, the same again, 4 MB in two batches,
# 64 MB, small ones after it.
for n, cap in ((1, 0), (10_000, 0), (20_000, 0), (20_000, 0), (62_500, 31_250), (1_000_000, 0),
               (1, 0), (20_000, 0), (1_000_000, 300_000)):
    call(n, cap)
g.free()
out.append(pinned()[1:])
print(json.dumps(out))
"""))
    *calls, end = got
    made, live, streams = ([c[k] for c in calls] for k in (2, 3, 4))
    assert made[0] <= 256 << 10 and made[1] <= 256 << 10 and made[2] <= 512 << 10
    assert made[3] == made[2]  # used again
    assert streams[0] == 1 and streams[4] == 2  # a second stream for a second batch
    assert max(live) <= 16 << 20 and made[5] <= 32 << 20
    assert made[5:] == [made[5]] * 4
    assert end == [0, 0]  # nothing left with the graph gone
