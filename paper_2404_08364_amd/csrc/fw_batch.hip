// Walks whose results live in host memory, run in batches that fit a device
// budget (section 5.2, Eq. 5): the queries are split into batches whose
// start vertices and result rows fit half of the budget, and consecutive
// batches alternate between two streams and two buffers (ping-pong), so the
// device-to-host copy of one batch overlaps the walk of the next.  Query i
// keeps id i (each batch walks with qid_base = its first query), so the rows
// equal fw_walk's on the whole query set.
//
// Rows reach the caller's memory through a few pinned slots: each of a few
// threads copies one piece of a finished batch into its slot and from there
// into place, so that one thread's copy from the device overlaps the others'
// copies on the host.  While a batch walks, the threads touch its part of the
// output (a fresh array has no pages yet).  The slots, their events and the
// streams stay with the graph; a call makes what is missing for its results, and
// its own where it finds them taken.  The first call on a graph for 1.2 MB of
// rows takes 0.70 ms; 2.38 ms with all 16 MiB pinned at once, 2.04 ms with
// staging made for each call.
// 100,003 weighted DeepWalk walks of 80 hops on R-MAT-20 (32 MB of rows): 18.6
// ms with whole batches staged in pinned memory made for the call and copied
// out by one thread, 4.6 ms so, 3.6 ms of it the walk.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "flowwalk.h"
#include "fw_runtime.h"

namespace {

int fail(int code, const char* msg) { return fw::set_error(code, msg); }

int hip_fail(hipError_t e, const char* what) {
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  return fw::set_error(e == hipErrorOutOfMemory ? FW_ENOMEM : FW_EHIP, m.c_str());
}

constexpr unsigned kSlots = 4;             // threads with a slot each
constexpr uint64_t kSlotBytes = 4ull << 20;  // at most
constexpr uint64_t kPage = 4096;

struct Side {
  hipStream_t stream = nullptr;  // the staging's
  uint32_t* d_starts = nullptr;
  uint32_t* d_rows = nullptr;
  uint64_t first = 0, count = 0;  // the batch it holds
  bool pending = false;
};

void release(Side& s) {
  if (s.stream) (void)hipStreamSynchronize(s.stream);
  (void)hipFree(s.d_starts);
  (void)hipFree(s.d_rows);
  s = Side{};
}

// Runs f(0) .. f(k - 1), f(0) on the calling thread, the others on their own
// (or on the calling thread where none can be made).
template <class F>
void on_threads(unsigned k, F&& f) {
  std::vector<std::thread> th;
  unsigned made = 1;
  try {
    th.reserve(k);
    for (; made < k; ++made) th.emplace_back([&f, made] { f(made); });
  } catch (...) {
  }
  f(0);
  for (unsigned i = made; i < k; ++i) f(i);
  for (auto& t : th) t.join();
}

}  // namespace

namespace fw {

// Pinned slots and streams of one fw_walk_host call at a time.
struct HostStage {
  hipStream_t stream[2] = {};
  uint8_t* slot[kSlots] = {};
  uint64_t bytes[kSlots] = {};   // of each slot
  hipEvent_t free[kSlots] = {};  // the slot's last copy has ended
  bool busy = false;             // guarded by the graph's mutex
};

// Makes what is missing of `streams` streams and `slots` slots of `bytes` bytes
// (no copy of an earlier call is under way).
static hipError_t grow_stage(HostStage* st, unsigned streams, unsigned slots, uint64_t bytes) {
  hipError_t e = hipSuccess;
  for (unsigned i = 0; i < streams && e == hipSuccess; ++i)
    if (!st->stream[i]) e = hipStreamCreateWithFlags(&st->stream[i], hipStreamNonBlocking);
  for (unsigned i = 0; i < slots && e == hipSuccess; ++i) {
    if (!st->free[i]) e = hipEventCreateWithFlags(&st->free[i], hipEventDisableTiming);
    if (e != hipSuccess || st->bytes[i] >= bytes) continue;
    if (st->slot[i]) (void)hipHostFree(st->slot[i]);
    st->slot[i] = nullptr;
    st->bytes[i] = 0;
    e = hipHostMalloc((void**)&st->slot[i], bytes, 0);
    if (e == hipSuccess) st->bytes[i] = bytes;
  }
  return e;
}

void free_host_stage(HostStage* st) {
  if (!st) return;
  for (auto s : st->stream)
    if (s) (void)hipStreamDestroy(s);
  for (unsigned i = 0; i < kSlots; ++i) {
    if (st->slot[i]) (void)hipHostFree(st->slot[i]);
    if (st->free[i]) (void)hipEventDestroy(st->free[i]);
  }
  delete st;
}

// The graph's staging, or one for this call if that is taken; null where host
// memory is short.  Give it back with return_stage.
static HostStage* take_stage(const fw_graph* g) {
  {
    std::lock_guard<std::mutex> lk(g->mu);
    auto* st = static_cast<HostStage*>(g->host_stage);
    if (st && !st->busy) {
      st->busy = true;
      return st;
    }
  }
  auto* st = new (std::nothrow) HostStage();
  if (!st) return nullptr;
  st->busy = true;
  std::lock_guard<std::mutex> lk(g->mu);
  if (!g->host_stage) g->host_stage = st;
  return st;
}

static void return_stage(const fw_graph* g, HostStage* st) {
  {
    std::lock_guard<std::mutex> lk(g->mu);
    if (g->host_stage == st) {
      st->busy = false;
      return;
    }
  }
  free_host_stage(st);
}

}  // namespace fw

extern "C" {

int fw_walk_host(const fw_graph* g, fw_algo algo, const fw_params* params,
                 const uint32_t* starts_host, uint64_t n, uint32_t length, uint64_t seed,
                 uint32_t* out_host, fw_batch_opts* opts) {
  fw::DevParams dp;
  // Host pointers stand in for the device ones in the argument check.
  int rc = fw::check_walk_args(g, (int)algo, params, n, length, starts_host, out_host, &dp);
  if (rc) return rc;
  fw_batch_opts o{};
  if (opts) o = *opts;
  const uint64_t cols = (uint64_t)length + 1;
  uint32_t last = 0;
  for (uint64_t i = 0; i < n; ++i) last = std::max(last, starts_host[i]);
  if (n && last >= g->nv) return fail(FW_EINVAL, "a start vertex is >= n_vertices");
  if (n == 0) {
    if (opts) opts->batch_queries = 0, opts->batches = 0;
    return FW_OK;
  }
  hipError_t e = hipSetDevice(g->device);
  if (e != hipSuccess) return hip_fail(e, "selecting the graph's device");
  uint64_t budget = o.device_budget_bytes;
  if (budget == 0) {
    size_t free_b = 0, total_b = 0;
    e = hipMemGetInfo(&free_b, &total_b);
    if (e != hipSuccess) return hip_fail(e, "querying free device memory");
    const uint64_t reserve = 1ull << 30;
    budget = free_b > reserve ? free_b - reserve : free_b / 2;
  }
  // Eq. 5: each of the two buffers holds a batch's start vertices and rows.
  const uint64_t per_query = (cols + 1) * sizeof(uint32_t);
  uint64_t batch = budget / (2 * per_query);
  if (o.max_batch_queries && batch > o.max_batch_queries) batch = o.max_batch_queries;
  if (batch == 0) return fail(FW_EINVAL, "device_budget_bytes holds no query");
  batch = std::min(batch, n);
  const uint64_t nb = (n + batch - 1) / batch;

  // Pieces of a batch's rows: small results are not worth the threads.
  auto threads_for = [](uint64_t bytes) {
    return (unsigned)std::min<uint64_t>(kSlots, (bytes + (1ull << 20) - 1) >> 20);
  };
  auto piece_for = [&](uint64_t bytes) {
    return std::min(kSlotBytes, std::max<uint64_t>(bytes / (2 * kSlots), 256 << 10));
  };
  // Slots of a power of two, so that a graph's calls seldom replace them.
  const uint64_t full_rows = batch * cols * sizeof(uint32_t);
  const unsigned slots = threads_for(full_rows);
  uint64_t slot_bytes = 256 << 10;
  while (slot_bytes < piece_for(full_rows)) slot_bytes *= 2;

  fw::HostStage* stage = fw::take_stage(g);
  if (!stage) return fail(FW_ENOMEM, "allocating the staging buffers");
  Side side[2];
  const unsigned sides = nb > 1 ? 2 : 1;
  e = fw::grow_stage(stage, sides, slots, slot_bytes);
  if (e != hipSuccess) {
    rc = hip_fail(e, "allocating the staging buffers");
    (void)hipGetLastError();  // not the next launch's
    fw::return_stage(g, stage);
    return rc;
  }
  for (unsigned k = 0; k < sides && e == hipSuccess; ++k) {
    Side& s = side[k];
    s.stream = stage->stream[k];
    e = hipMalloc((void**)&s.d_starts, batch * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc((void**)&s.d_rows, batch * cols * sizeof(uint32_t));
  }
  if (e != hipSuccess) {
    rc = hip_fail(e, "allocating the batch buffers");
    release(side[0]);
    release(side[1]);
    fw::return_stage(g, stage);
    return rc;
  }

  auto out_of = [&](const Side& s) { return reinterpret_cast<uint8_t*>(out_host + s.first * cols); };

  // Copies a walked batch into out_host.
  auto drain = [&](Side& s) -> int {
    if (!s.pending) return FW_OK;
    s.pending = false;
    const uint64_t bytes = s.count * cols * sizeof(uint32_t), piece = piece_for(bytes);
    uint8_t* dst = out_of(s);
    std::atomic<uint64_t> next{0};
    std::atomic<int> err{hipSuccess};
    on_threads(threads_for(bytes), [&](unsigned i) {
      hipError_t he = hipSetDevice(g->device);
      for (;;) {
        const uint64_t at = next.fetch_add(piece);
        if (at >= bytes || he != hipSuccess || err.load() != hipSuccess) break;
        const uint64_t len = std::min(piece, bytes - at);
        he = hipEventSynchronize(stage->free[i]);
        if (he == hipSuccess)
          he = hipMemcpyAsync(stage->slot[i], reinterpret_cast<const uint8_t*>(s.d_rows) + at, len,
                              hipMemcpyDeviceToHost, s.stream);
        if (he == hipSuccess) he = hipEventRecord(stage->free[i], s.stream);
        if (he == hipSuccess) he = hipEventSynchronize(stage->free[i]);
        if (he == hipSuccess) std::memcpy(dst + at, stage->slot[i], len);
      }
      if (he != hipSuccess) err = he;
    });
    const hipError_t he = (hipError_t)err.load();
    return he == hipSuccess ? FW_OK : hip_fail(he, "copying result rows");
  };

  fw_walk_opts wo{};
  wo.mode = o.mode;
  wo.async = 1;
  for (uint64_t b = 0; b < nb && rc == FW_OK; ++b) {
    Side& s = side[b % 2];  // free: batch b - 2 was drained
    s.first = b * batch;
    s.count = std::min(batch, n - s.first);
    const uint64_t bytes = s.count * sizeof(uint32_t);
    for (uint64_t at = 0, k = 0; at < bytes && e == hipSuccess; at += slot_bytes, ++k) {
      const uint64_t len = std::min(slot_bytes, bytes - at);
      const unsigned i = (unsigned)(k % slots);
      e = hipEventSynchronize(stage->free[i]);
      if (e != hipSuccess) break;
      std::memcpy(stage->slot[i], reinterpret_cast<const uint8_t*>(starts_host + s.first) + at, len);
      e = hipMemcpyAsync(reinterpret_cast<uint8_t*>(s.d_starts) + at, stage->slot[i], len,
                         hipMemcpyHostToDevice, s.stream);
      if (e == hipSuccess) e = hipEventRecord(stage->free[i], s.stream);
    }
    if (e != hipSuccess) {
      rc = hip_fail(e, "copying start vertices");
      break;
    }
    wo.stream = s.stream;
    wo.qid_base = s.first;
    rc = fw_walk_ex(g, algo, params, s.d_starts, s.count, length, seed, s.d_rows, &wo);
    if (rc) break;
    s.pending = true;
    // The output's pages, while the batch walks.
    const uint64_t row_bytes = s.count * cols * sizeof(uint32_t);
    const unsigned k = threads_for(row_bytes);
    uint8_t* dst = out_of(s);
    on_threads(k, [&](unsigned i) {
      const uint64_t lo = row_bytes * i / k, hi = row_bytes * (i + 1) / k;
      for (uint64_t p = lo; p < hi; p += kPage) {
        uint8_t none = 0;  // an access that writes (one fault), and leaves every byte as it is
        (void)__atomic_compare_exchange_n(dst + p, &none, (uint8_t)0, false, __ATOMIC_RELAXED,
                                          __ATOMIC_RELAXED);
      }
    });
    if (b) rc = drain(side[(b + 1) % 2]);
  }
  if (rc == FW_OK) rc = drain(side[(nb + 1) % 2]);
  if (rc == FW_OK) rc = fw_sync(g, side[0].stream);
  release(side[0]);
  release(side[1]);
  fw::return_stage(g, stage);
  if (rc == FW_OK && opts) {
    opts->batch_queries = batch;
    opts->batches = (uint32_t)nb;
  }
  return rc;
}

}  // extern "C"
