// Request access of the dynamically scheduled walkers.
#pragma once

#include "fw_kernels.h"

namespace fw {

// Claims of one wavefront from a launch's head counter, which counts the
// queries past the wavefronts' first ones.  Atomics on it run one after the
// other, about 11 ns each over the chip, so a wavefront whose claims follow
// each other faster than all wavefronts can have one each doubles what it
// takes, and halves it again when they are far apart: one or two queries of
// long walks, up to 64 of short ones, and at most half its share of what is
// left, so that the last claims are small.  Against claims of an eighth of the
// share, at least one query per empty group: 300,000 PPR walks on R-MAT-18
// 1.72 and 0.85 ms, 1,048,576 from the hub of R-MAT-22 5.72 and 4.98 ms (10.3
// with an atomic per round), 2,097,152 MetaPath walks of 20 hops on Chung-Lu
// 2^22 15.2 and 14.6 ms; walks of 80 hops within 3 % on all sizes.
struct Claims {
  static constexpr uint32_t kMaxClaim = 64;
  uint64_t since;  // when the last claim (or the launch) began, 10 ns ticks
  uint32_t last;   // queries it was for

  __device__ __forceinline__ Claims() : since(__builtin_amdgcn_s_memrealtime()), last(1) {}

  // Claims queries [lo, hi) of those before n, at least `least`; first: the
  // queries that are not the counter's.  hi comes in as the end of the last
  // claim.  Returns false (and lo = hi = n) when none are left.
  __device__ __forceinline__ bool next(uint64_t* __restrict__ head, uint64_t first, uint64_t n,
                                       uint64_t waves, uint32_t least, uint64_t& lo,
                                       uint64_t& hi) {
    const uint64_t now = __builtin_amdgcn_s_memrealtime();
    const uint64_t ticks = now - since;  // about `waves` ticks let every wavefront claim once
    const uint32_t share = (uint32_t)min((n - hi) / (2 * waves), (uint64_t)kMaxClaim);
    uint32_t k = ticks < 2 * waves ? 2 * last : ticks > 4 * waves ? last / 2 : last;
    k = max(min(k, share), least);
    uint64_t at = 0;
    if (lane_id() == 0) at = atomicAdd((unsigned long long*)head, (unsigned long long)k);
    lo = min(first + readlane64(at, 0), n);
    hi = min(lo + k, n);
    since = now;
    last = k;
    return lo < n;
  }
};

// Request access: a single request passed by value, or a table of requests
// (binary search of the query-count prefix maps a global index to its
// request).
template <bool MULTI>
struct Reqs {
  ReqDesc one;
  ReqTable tab;
  __device__ __forceinline__ uint64_t total() const { return MULTI ? tab.total : one.n; }
  __device__ __forceinline__ uint32_t find(uint64_t q) const {
    if (!MULTI) return 0;
    uint32_t lo = 0, hi = tab.nreq;  // last r with prefix[r] <= q
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) / 2;
      if (tab.prefix[mid] <= q)
        lo = mid;
      else
        hi = mid;
    }
    return lo;
  }
  __device__ __forceinline__ uint64_t first(uint32_t r) const {
    return MULTI ? tab.prefix[r] : 0;
  }
  __device__ __forceinline__ ReqDesc get(uint32_t r) const { return MULTI ? tab.reqs[r] : one; }
};

// Served form: a retired query adds its realised hops to its request's
// counter (one atomic per query).
__device__ __forceinline__ void count_steps(const ReqDesc& R, uint32_t hops) {
  if (R.steps != nullptr && hops != 0) atomicAdd(R.steps, (unsigned long long)hops);
}

// Enqueues the reset of a launch's head counter.
hipError_t reset_counter(uint64_t* head, hipStream_t stream);

// Walks of unweighted DeepWalk and PPR (fw_uniform.hip), at most wgs_per_cu
// 256-thread workgroups per CU; resets `head` where it is used.
template <bool MULTI>
hipError_t launch_uniform(int algo, const DevGraph& g, const Reqs<MULTI>& rq, uint32_t* status,
                          uint64_t* head, int num_cus, uint32_t wgs_per_cu, uint64_t n,
                          hipStream_t stream);

}  // namespace fw
