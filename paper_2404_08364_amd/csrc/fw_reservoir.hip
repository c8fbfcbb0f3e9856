// Reservoir-sampling walkers (section 4): the paper's two parallel reservoir
// samplers as alternatives to the inverse-CDF pick, one wavefront per query
// (claimed from a head counter: rows of very different lengths leave a static
// assignment waiting for its longest wavefront).
//
// Each entry i of the hop's neighbour sequence gets its own uniform word:
// word i mod 4 of Philox4x64-10 at counter (qid, t, i / 4, 1), key (seed, 0).
// Lane L handles quads of four consecutive entries.  Visiting entry i of
// weight w_i with W the running total including it, the selection becomes i
// when floor(u_i * W / 2^64) < w_i (the integer form of "random(0,1) <
// w_i / W"); the last selection is the pick.
//
//   DPRS (Algorithm 3): 256-entry chunks in sequence order (lane L holds
//   quad 64c + L); per chunk one wave scan gives each entry its running total
//   and one ballot keeps the last selection.  The result is that of the
//   sequential reservoir over S.  Where weights are cheap to read (all but
//   node2vec) the chunks are visited from the last one (dprs_pick_back).
//   ZPRS (Algorithm 4): lane L owns quads L, L + 64, ... ; pass 1 sums each
//   lane's weights, an exclusive wave scan gives each lane its starting
//   total, pass 2 re-reads the lane's quads and selects along the zig-zag
//   order S' (lane 0's entries, then lane 1's, ...); the last lane holding a
//   selection wins.
// Node2vec membership is the binary search of N(prev) in global memory, as
// the paper's samplers do it.
#include "fw_kernels.h"
#include "fw_requests.h"
#include "fw_reservoir.h"

namespace fw {

// Relative quads of a row for dprs_pick_back (DeepWalk, PPR, MetaPath).  Rows
// start at any entry, so a quad is read as four 4-byte words in one 16-byte
// load; the arrays are padded by more than a quad.
template <int ALGO, bool WEIGHTED>
struct RowQuads {
  struct Words4 {
    uint32_t v[4];
  };
  struct Loaded {
    Words4 w;
    uint32_t l;
  };
  const uint32_t* __restrict__ w;    // the row's weights
  const uint8_t* __restrict__ lab;   // and labels
  uint32_t d, want;

  __device__ __forceinline__ Loaded load(uint32_t q) const {
    const uint32_t last = (d - 1) / 4;
    q = q < last ? q : last;
    Loaded v{{{1u, 1u, 1u, 1u}}, 0u};
    if (WEIGHTED) __builtin_memcpy(&v.w, w + 4ull * q, sizeof(v.w));
    if (ALGO == kMetaPath) __builtin_memcpy(&v.l, lab + 4ull * q, sizeof(v.l));
    return v;
  }
  __device__ __forceinline__ void weights(const Loaded& v, uint32_t q, uint32_t out[4]) const {
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      bool in = 4 * q + j < d;
      if (ALGO == kMetaPath) in = in && ((v.l >> (8 * j)) & 0xFFu) == want;
      out[j] = in ? v.w.v[j] : 0u;
    }
  }
  __device__ __forceinline__ uint64_t total(uint32_t quads) const {
    if (ALGO != kMetaPath && !WEIGHTED) return d;
    uint64_t acc = 0;
#pragma unroll 1
    for (uint32_t q = (uint32_t)lane_id(); q < quads + (uint32_t)lane_id(); q += 4 * kWave) {
      Loaded v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = load(q + k * kWave);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        uint32_t x[4];
        weights(v[k], q + k * kWave, x);
        acc += ((uint64_t)x[0] + x[1]) + ((uint64_t)x[2] + x[3]);
      }
    }
    return wave_sum(acc);
  }
};

template <int ALGO, bool WEIGHTED, bool ZIGZAG>
__global__ __launch_bounds__(256) void k_walk_reservoir(DevGraph g, DevParams prm,
                                                        const uint32_t* __restrict__ starts,
                                                        uint64_t n, uint32_t length,
                                                        uint64_t seed, uint64_t qid_base,
                                                        uint32_t* __restrict__ out,
                                                        uint32_t* __restrict__ status,
                                                        uint64_t* __restrict__ head) {
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
  const int lane = lane_id();
  // The first query by the wavefront's index, later ones from the head
  // counter, an eighth of the wavefront's share of what is left at a time.
  uint64_t q = uniform64(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave);
  uint64_t q_end = q + 1;
  for (;; ++q) {
    if (q == q_end) {
      if (nwaves >= n) break;
      uint64_t k = (n - min(q, n)) / (nwaves * 8);
      k = k < 1 ? 1 : k > kMaxClaim ? kMaxClaim : k;
      uint64_t base = 0;
      if (lane == 0) base = atomicAdd((unsigned long long*)head, (unsigned long long)k);
      q = nwaves + readlane64(base, 0);
      q_end = q + k;
    }
    if (q >= n) break;
    const uint32_t s = uniform32(starts[q]);
    uint32_t* row = out + q * ((uint64_t)length + 1);
    if (s >= g.nv) {
      if (lane == 0) atomicOr(status, 1u);
      continue;
    }
    if (lane == 0) row[0] = s;
    const uint64_t qid = qid_base + q;
    uint32_t cur = s, prev = kEnd, t = 0;
    for (; t < length; ++t) {
      if (ALGO == kPPR && ppr_stops(prm, seed, qid, t)) break;
      const uint64_t o = g.off[cur];
      const uint64_t d = g.off[cur + 1] - o;
      Eval<ALGO, WEIGHTED> ev;
      ev.adj = g.adj;
      ev.w = g.w;
      ev.lab = g.lab;
      ev.o = o;
      ev.first = (t == 0);
      ev.prev = prev;
      ev.f_ret = prm.f_ret;
      ev.f_in = prm.f_in;
      ev.f_out = prm.f_out;
      ev.mem.adj = g.adj;
      ev.mem.po = ev.mem.pd = 0;
      if (ALGO == kNode2Vec && t > 0) {
        ev.mem.po = g.off[prev];
        ev.mem.pd = g.off[prev + 1] - ev.mem.po;
      }
      ev.want = (ALGO == kMetaPath) ? schema_label(prm, t) : 0u;
      int64_t idx;
      if constexpr (ZIGZAG)
        idx = zprs_pick(ev, d, seed, qid, t);
      else if constexpr (ALGO == kNode2Vec)  // a weight costs a search: read once
        idx = dprs_pick(ev, d, seed, qid, t);
      else
        idx = d == 0 ? -1
                     : dprs_pick_back(RowQuads<ALGO, WEIGHTED>{g.w + o, g.lab + o, (uint32_t)d,
                                                               ev.want},
                                      (uint32_t)d, seed, qid, t);
      if (idx < 0) break;
      const uint32_t nxt = uniform32(g.adj[o + (uint64_t)idx]);
      if (lane == 0) row[t + 1] = nxt;
      prev = cur;
      cur = nxt;
    }
    for (uint32_t p = t + 1 + lane; p <= length; p += kWave) row[p] = kEnd;
  }
}

hipError_t launch_reservoir(const LaunchArgs& a, int sampler, hipStream_t stream) {
  const int block = 256;
  uint64_t blocks = (a.n + (block / kWave) - 1) / (block / kWave);
  const uint64_t cap = (uint64_t)a.num_cus * 8;  // what is resident at a time
  if (blocks > cap) blocks = cap;
  if (blocks == 0) blocks = 1;
  if (blocks * (block / kWave) < a.n) {  // only then is the counter claimed from
    const hipError_t e = reset_counter(a.head, stream);
    if (e != hipSuccess) return e;
  }
  const bool wt = a.g.w != nullptr;
  const bool zz = sampler == 2;
#define FW_GO(A, W, Z)                                                                          \
  hipLaunchKernelGGL((k_walk_reservoir<A, W, Z>), dim3((unsigned)blocks), dim3(block), 0,       \
                     stream, a.g, a.prm, a.starts, a.n, a.length, a.seed, a.qid_base, a.out,     \
                     a.status, a.head)
#define FW_GO2(A)                                 \
  if (wt) {                                       \
    if (zz) FW_GO(A, true, true); else FW_GO(A, true, false);   \
  } else {                                        \
    if (zz) FW_GO(A, false, true); else FW_GO(A, false, false); \
  }
  switch (a.algo) {
    case kDeepWalk: FW_GO2(kDeepWalk); break;
    case kNode2Vec: FW_GO2(kNode2Vec); break;
    case kMetaPath: FW_GO2(kMetaPath); break;
    case kPPR: FW_GO2(kPPR); break;
    default:
      return hipErrorInvalidValue;
  }
#undef FW_GO2
#undef FW_GO
  return hipGetLastError();
}

}  // namespace fw
