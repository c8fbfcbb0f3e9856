// Reservoir-sampling walkers (section 4): the paper's two parallel reservoir
// samplers as alternatives to the inverse-CDF pick, one wavefront per query
// (one workgroup per query, handed out by the dispatcher).
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
//   sequential reservoir over S.  The chunks are visited from the last one
//   (dprs_pick_back).
//   ZPRS (Algorithm 4): lane L owns quads L, L + 64, ... ; pass 1 sums each
//   lane's weights, an exclusive wave scan gives each lane its starting
//   total, pass 2 re-reads the lane's quads and selects along the zig-zag
//   order S' (lane 0's entries, then lane 1's, ...); the last lane holding a
//   selection wins.
// Node2vec membership is an LDS hash set of N(prev), or a binary search of its
// row where that is long, for the four entries of a quad at once.
#include <algorithm>

#include "fw_kernels.h"
#include "fw_member.h"
#include "fw_reservoir.h"

namespace fw {

// LDS cells of a wavefront's hash set of N(prev).
constexpr uint32_t kSetCells = 1024;

template <int ALGO>
struct WeightOf {
  using type = uint32_t;
};
template <>
struct WeightOf<kNode2Vec> {
  using type = uint64_t;  // weight times factor
};

// Relative quads of a row for the pickers.  Rows start at any entry, so a quad
// is read as four 4-byte words in one 16-byte load; the arrays are padded by
// more than a quad.  1,394 node2vec walks of 10 hops with DPRS on R-MAT-16:
// 260 us with a binary search per entry, one after the other, 129 us with the
// hash set; 40,000 on R-MAT-19 4.87 and 2.11 ms.
template <int ALGO, bool WEIGHTED>
struct RowQuads {
  using Weight = typename WeightOf<ALGO>::type;
  struct Words4 {
    uint32_t v[4];
  };
  struct Loaded {
    Words4 w, a;  // weights; node2vec past the first hop: ids
    uint32_t l;   // MetaPath: labels
  };
  const uint32_t* __restrict__ w;    // the row's weights,
  const uint32_t* __restrict__ adj;  // ids
  const uint8_t* __restrict__ lab;   // and labels
  uint32_t d, want;
  // node2vec (Eq. 2).
  MemberAny mem;
  uint32_t prev, f_ret, f_in, f_out;
  bool first;

  __device__ __forceinline__ Loaded load(uint32_t q) const {
    const uint32_t last = (d - 1) / 4;
    q = q < last ? q : last;
    Loaded v{{{1u, 1u, 1u, 1u}}, {{0u, 0u, 0u, 0u}}, 0u};
    if (WEIGHTED) __builtin_memcpy(&v.w, w + 4ull * q, sizeof(v.w));
    if (ALGO == kNode2Vec && !first) __builtin_memcpy(&v.a, adj + 4ull * q, sizeof(v.a));
    if (ALGO == kMetaPath) __builtin_memcpy(&v.l, lab + 4ull * q, sizeof(v.l));
    return v;
  }
  __device__ __forceinline__ void weights(const Loaded& v, uint32_t q, Weight out[4]) const {
    uint32_t f[4] = {1u, 1u, 1u, 1u};
    if (ALGO == kNode2Vec && !first) {
      mem.factors4(v.a.v, f_in, f_out, f);
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = v.a.v[j] == prev ? f_ret : f[j];
    }
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      bool in = 4 * q + j < d;
      if (ALGO == kMetaPath) in = in && ((v.l >> (8 * j)) & 0xFFu) == want;
      out[j] = in ? (Weight)v.w.v[j] * f[j] : (Weight)0;
    }
  }
  __device__ __forceinline__ uint64_t total(uint32_t quads) const {
    if (ALGO != kMetaPath && !WEIGHTED && (ALGO != kNode2Vec || first)) return d;
    if (ALGO == kNode2Vec && !first) {  // the lookups are what takes the time
      uint64_t acc = 0;
#pragma unroll 1
      for (uint32_t c = 0; c < quads; c += kWave) {
        const uint32_t q = c + (uint32_t)lane_id();
        Weight x[4];
        weights(load(q), q, x);
        acc += (x[0] + x[1]) + (x[2] + x[3]);
      }
      return wave_sum(acc);
    }
    uint64_t acc = 0;
#pragma unroll 1
    for (uint32_t q = (uint32_t)lane_id(); q < quads + (uint32_t)lane_id(); q += 4 * kWave) {
      Loaded v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = load(q + k * kWave);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        Weight x[4];
        weights(v[k], q + k * kWave, x);
        acc += ((uint64_t)x[0] + x[1]) + ((uint64_t)x[2] + x[3]);
      }
    }
    return wave_sum(acc);
  }
};

template <int ALGO, bool WEIGHTED, bool ZIGZAG>
__global__ __launch_bounds__(kWave) void k_walk_reservoir(DevGraph g, DevParams prm,
                                                        const uint32_t* __restrict__ starts,
                                                        uint64_t n, uint32_t length,
                                                        uint64_t seed, uint64_t qid_base,
                                                        uint32_t* __restrict__ out,
                                                        uint32_t* __restrict__ status) {
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
  const int lane = lane_id();
  for (uint64_t q = uniform64(wave); q < n; q += nwaves) {
    const uint32_t s = uniform32(starts[q]);
    uint32_t* row = out + q * ((uint64_t)length + 1);
    if (s >= g.nv) {
      if (lane == 0) flag_bad_start(status);
      continue;
    }
    if (lane == 0) row[0] = s;
    const uint64_t qid = qid_base + q;
    uint32_t cur = s, prev = kEnd, t = 0;
    uint64_t po = 0, pd = 0;
    for (; t < length; ++t) {
      if (ALGO == kPPR && ppr_stops(prm, seed, qid, t)) break;
      const uint64_t o = g.off[cur];
      const uint64_t d = g.off[cur + 1] - o;
      int64_t idx = -1;
      if (d != 0) {
        RowQuads<ALGO, WEIGHTED> rq;
        rq.w = g.w + o;
        rq.adj = g.adj + o;
        rq.lab = g.lab + o;
        rq.d = (uint32_t)d;
        rq.want = (ALGO == kMetaPath) ? schema_label(prm, t) : 0u;
        rq.first = t == 0;
        if (ALGO == kNode2Vec) {
          rq.prev = prev;
          rq.f_ret = prm.f_ret;
          rq.f_in = prm.f_in;
          rq.f_out = prm.f_out;
          Table tb;
          tb.cells = kSetCells;
          tb.base = (threadIdx.x / kWave) * kSetCells;
          tb.po = po;
          tb.pd = t == 0 ? 0 : pd;
          build_table(tb, g.adj, d, lane, false);
          rq.mem.mode = tb.kind;
          rq.mem.base = tb.base;
          rq.mem.bmask = tb.bmask;
          rq.mem.shift = tb.shift;
          rq.mem.adj = g.adj;
          rq.mem.po = tb.po;
          rq.mem.pd = tb.pd;
        }
        idx = ZIGZAG ? zprs_pick_row(rq, (uint32_t)d, seed, qid, t)
                     : dprs_pick_back(rq, (uint32_t)d, seed, qid, t);
        wave_sync_lds();
      }
      if (idx < 0) break;
      const uint32_t nxt = uniform32(g.adj[o + (uint64_t)idx]);
      if (lane == 0) row[t + 1] = nxt;
      prev = cur;
      cur = nxt;
      po = o;  // the next hop's N(prev)
      pd = d;
    }
    for (uint32_t p = t + 1 + lane; p <= length; p += kWave) row[p] = kEnd;
  }
}

hipError_t launch_reservoir(const LaunchArgs& a, int sampler, hipStream_t stream) {
  // One wavefront per workgroup and one query per wavefront: the dispatcher
  // hands a free slot the next query at no cost to the walks.  (Rows of very
  // different lengths leave a static share of the queries waiting for its
  // longest wavefront, and claims from a counter cost an atomic of about 12 ns
  // each, one after the other over the chip: 40,000 MetaPath walks of 10 hops
  // on R-MAT-16 289 us with a static share, 545 us with claims, 201 us so.)
  const int block = kWave;
  const uint64_t blocks = std::max<uint64_t>(1, std::min<uint64_t>(a.n, 1ull << 22));
  const bool wt = a.g.w != nullptr;
  const bool zz = sampler == 2;
#define FW_GO(A, W, Z)                                                                          \
  hipLaunchKernelGGL((k_walk_reservoir<A, W, Z>), dim3((unsigned)blocks), dim3(block),          \
                     A == kNode2Vec ? block / kWave * kSetCells * sizeof(uint32_t) : 0, stream,    \
                     a.g, a.prm, a.starts, a.n, a.length, a.seed, a.qid_base, a.out, a.status)
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
