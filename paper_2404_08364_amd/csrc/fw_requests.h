// Request access of the dynamically scheduled walkers.
#pragma once

#include "fw_kernels.h"

namespace fw {

// Queries claimed at a time, at most.  1,048,576 PPR walks from the hub of
// R-MAT-22 took 10.3 ms with one atomic per round that emptied a group, 6.2 ms
// with claims of up to 32 that shrink towards the end.
constexpr uint64_t kMaxClaim = 32;

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
