// Walker of unweighted DeepWalk and PPR: one query per lane.
//
// With unit weights the total of a row is its degree and the prefix sum at
// entry i is i + 1, so the pick of the exact inverse CDF is the draw itself,
// r = floor(u * d / 2^64), and a hop reads two offsets and one id whatever
// the degree.  Nothing is left for a wavefront to share: each lane walks its
// own query, and the 64 dependent chains of a wavefront (offsets, then the
// id) overlap.  The bound is the rate of scattered cache-line reads, so the
// grid fills every SIMD with eight wavefronts.  One million walks of 80 hops
// on R-MAT-21 (47.4 M hops): 65.9 ms with a wavefront per hop summing the
// row's unit weights, 1.61 ms here.
//
// Rows: a lane collects 16 consecutive entries in LDS (entry p at
// [p mod 16][lane], conflict-free) and stores them as four 16-byte words;
// the tail of a row that ended early is filled by the whole wavefront.
#include "fw_kernels.h"
#include "fw_requests.h"

namespace fw {

namespace {

constexpr int kBlock = 256;
constexpr uint32_t kRun = 16;  // entries per store run
// Empty lanes that make a claim worth its atomic's latency (a PPR walk of
// stop chance 1/5 empties about 12 lanes of a wavefront per hop).
constexpr uint32_t kClaimMin = 16;

struct alignas(4) Words4 {
  uint32_t v[4];
};

// Entries [p - p mod 16, p] of the lane's row, from its LDS run.
__device__ __forceinline__ void store_run(uint32_t* row, const uint32_t* run, uint32_t p) {
  const uint32_t b = p & ~(kRun - 1);
  if (p - b == kRun - 1) {
#pragma unroll
    for (uint32_t k = 0; k < kRun; k += 4) {
      Words4 w;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) w.v[j] = run[(k + j) * kWave];
      __builtin_memcpy(row + b + k, &w, sizeof(w));
    }
  } else {
    for (uint32_t k = b; k <= p; ++k) row[k] = run[(k - b) * kWave];
  }
}

template <int ALGO, bool MULTI>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void
k_walk_uniform(DevGraph g, Reqs<MULTI> rq, uint32_t* __restrict__ status,
               uint64_t* __restrict__ head) {
  __shared__ uint32_t runs[kBlock / kWave][kRun * kWave];
  const int lane = lane_id();
  uint32_t* run = &runs[threadIdx.x / kWave][lane];
  const uint64_t n = rq.total();
  const uint64_t lanes = (uint64_t)gridDim.x * kBlock;

  uint32_t* row = nullptr;
  uint64_t seed = 0, qid = 0;
  uint32_t cur = 0, t = 0, length = 0, req = 0;
  uint32_t stop_num = 0, stop_den = 1;
  bool live = false;
  // The first query of every lane is its own index; the head counter hands
  // out the ones past the grid.
  uint64_t pool = uniform64((uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~(uint32_t)(kWave - 1)));
  uint64_t pool_end = min(pool + kWave, n);
  pool = min(pool, n);
  bool exhausted = pool == n;
  Claims claims;

  for (;;) {
    if (!exhausted) {
      const uint64_t empty_m = ballot(!live);
      const uint32_t empty = (uint32_t)__builtin_popcountll(empty_m);
      if (empty >= kClaimMin) {
        if (pool == pool_end &&
            !claims.next(head, lanes, n, lanes / kWave, empty, pool, pool_end))
          exhausted = true;
        const uint64_t base = pool;
        if (!live) {
          const uint64_t q = base + (uint32_t)__builtin_popcountll(empty_m & ((1ull << lane) - 1));
          if (q < pool_end) {
            req = rq.find(q);
            const ReqDesc R = rq.get(req);
            const uint64_t lq = q - rq.first(req);
            cur = R.starts[lq];
            if (cur >= g.nv) {
              flag_bad_start(status);
            } else {
              length = R.length;
              row = R.out + lq * ((uint64_t)length + 1);
              seed = R.seed;
              qid = R.qid_base + lq;
              stop_num = R.prm.stop_num;
              stop_den = R.prm.stop_den;
              t = 0;
              live = length > 0;
              if (live)
                run[0] = cur;
              else
                row[0] = cur;
            }
          }
        }
        pool = pool + empty < pool_end ? pool + empty : pool_end;
        if (pool == pool_end && (pool_end == n || n <= lanes)) exhausted = true;
      }
    }
    if (!ballot(live)) {
      if (exhausted) break;
      continue;
    }
    bool end = false;
    if (live) {
      const uint64_t o = g.off[cur];
      const uint64_t d = g.off[(uint64_t)cur + 1] - o;
      uint64_t word1;
      const uint64_t u = philox_draw2(seed, qid, t, word1);
      end = d == 0;
      if (ALGO == kPPR)
        end |= __umul64hi(word1, (uint64_t)stop_den) < (uint64_t)stop_num;
      if (!end) {
        cur = g.adj[o + scale_draw(u, d)];
        ++t;
        run[(t & (kRun - 1)) * kWave] = cur;
      }
      // A run is stored when it is full and when its row ends.
      const bool full = !end && (t & (kRun - 1)) == kRun - 1;
      const bool last = end ? (t & (kRun - 1)) != kRun - 1 : t == length;
      if (full || last) store_run(row, run, t);
      if (!end && t == length) live = false;
      if (MULTI && (end || !live)) {
        ReqDesc R = rq.get(req);
        count_steps(R, t);
      }
    }
    // Rows that ended early: FW_END up to their last entry.
    for (uint64_t m = ballot(end); m; m &= m - 1) {
      const int src = first_lane(m);
      uint32_t* r = reinterpret_cast<uint32_t*>(readlane64(reinterpret_cast<uint64_t>(row), src));
      const uint32_t len = readlane32(length, src);
      for (uint64_t p = (uint64_t)readlane32(t, src) + 1 + lane; p <= len; p += kWave) r[p] = kEnd;
    }
    if (end) live = false;
  }
}

template <int ALGO, bool MULTI>
hipError_t go(const DevGraph& g, const Reqs<MULTI>& rq, uint32_t* status, uint64_t* head,
              unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((k_walk_uniform<ALGO, MULTI>), dim3(blocks), dim3(kBlock), 0, stream, g, rq,
                     status, head);
  return hipGetLastError();
}

}  // namespace

template <bool MULTI>
hipError_t launch_uniform(int algo, const DevGraph& g, const Reqs<MULTI>& rq, uint32_t* status,
                          uint64_t* head, int num_cus, uint32_t wgs_per_cu, uint64_t n,
                          hipStream_t stream) {
  const uint64_t cap = (uint64_t)num_cus * wgs_per_cu;
  const uint64_t need = (n + kBlock - 1) / kBlock;
  const unsigned blocks = (unsigned)(need < cap ? need : cap);
  if (need > cap) {  // only then does a lane claim from the counter
    const hipError_t e = reset_counter(head, stream);
    if (e != hipSuccess) return e;
  }
  switch (algo) {
    case kDeepWalk: return go<kDeepWalk>(g, rq, status, head, blocks, stream);
    case kPPR: return go<kPPR>(g, rq, status, head, blocks, stream);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_uniform<false>(int, const DevGraph&, const Reqs<false>&, uint32_t*,
                                          uint64_t*, int, uint32_t, uint64_t, hipStream_t);
template hipError_t launch_uniform<true>(int, const DevGraph&, const Reqs<true>&, uint32_t*,
                                         uint64_t*, int, uint32_t, uint64_t, hipStream_t);

}  // namespace fw
