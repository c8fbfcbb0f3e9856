// Group totals of hub rows, kept in LDS for the length of a launch.
//
// Walks meet a vertex in proportion to its degree and a hop's first pass
// streams the whole row, so on power-law graphs a few rows take most of the
// traffic (the 300 longest rows of R-MAT-22 hold 56 % of the entries that
// walks scan, those of Chung-Lu 2^22, gamma 2.1, 93 %).  The first pass of
// an algorithm whose weights depend only on the vertex (and MetaPath's wanted
// label) leaves the same 64 group totals on every visit: the wavefronts of a
// workgroup share them here, and a later visit reads 64 words from LDS and
// one group of the row, 1/64 of it.  Measured on one MI355X, before and after:
// 524,288 weighted DeepWalk walks of 80 hops on R-MAT-22 48.8 and 35.8 ms,
// node2vec 142.4 and 137.9 ms (raw weight totals of the rows that take the
// regrouped pass; 15 buckets beside the membership regions), 1,048,576 PPR
// walks from its largest hub 24.8 and 10.4 ms, 2,097,152 MetaPath walks of 20
// hops on Chung-Lu 2^22 46.0 and 27.3 ms.
//
// Layout: buckets of four ways, each way a key (vertex, label), its degree
// and 64 totals of 32 bits (rows with a larger total are not kept).  A row
// replaces the shortest way of its bucket if that is shorter than itself, so
// a way's degree only grows; the top bit of the degree marks a way being
// written.  Readers never wait: they read the key, the totals and the key
// again.  A way that changed in between held another row of strictly larger
// degree meanwhile and cannot have got the old key back.
#pragma once

#include "fw_device.h"

namespace fw {

// Rows from this degree on are looked up and kept.
constexpr uint32_t kHubMinDegree = 2048;
constexpr uint32_t kHubWays = 4;
constexpr uint32_t kHubBusy = 0x80000000u;
// Words of a bucket: keys, labels, degrees, totals.
constexpr uint32_t kHubBucketWords = 3 * kHubWays + kHubWays * kWave;

using hub_ptr = __attribute__((address_space(3))) uint32_t*;

__device__ __forceinline__ uint32_t hub_load(hub_ptr p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void hub_store(hub_ptr p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Orders the wavefront's LDS accesses before against those after.
__device__ __forceinline__ void hub_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
}

// No cache: every first pass streams its row.
struct NoHubs {
  __device__ __forceinline__ bool find(uint32_t, uint64_t&) const { return false; }
  __device__ __forceinline__ void keep(uint32_t, uint64_t) const {}
};

// The cache as seen from one hop: its row's key.
struct Hubs {
  hub_ptr base;
  uint32_t buckets;  // 0: no cache
  uint32_t cur, want;

  __device__ __forceinline__ hub_ptr bucket() const {
    const uint32_t h = (cur ^ (want * 0x85EBCA6Bu)) * 0x9E3779B1u;
    return base + __umulhi(h, buckets) * kHubBucketWords;
  }
  __device__ __forceinline__ bool holds(hub_ptr b, uint32_t way) const {
    return hub_load(b + way) == cur && hub_load(b + kHubWays + way) == want;
  }

  // Lane g gets the total of group g of the row, if it is here.  (d: the
  // row's degree; every lane of the wavefront calls.)
  __device__ __forceinline__ bool find(uint32_t d, uint64_t& mine) const {
    if (buckets == 0 || d < kHubMinDegree) return false;
    const hub_ptr b = bucket();
    uint32_t way = kHubWays;
#pragma unroll
    for (uint32_t k = 0; k < kHubWays; ++k) way = holds(b, k) ? k : way;
    way = uniform32(way);
    if (way == kHubWays) return false;
    hub_fence();
    const uint32_t tot = hub_load(b + 3 * kHubWays + way * kWave + (uint32_t)lane_id());
    hub_fence();
    if (!uniform32(holds(b, way) ? 1u : 0u)) return false;
    mine = tot;
    return true;
  }

  // Offers the row's totals (lane g: group g's).
  __device__ __forceinline__ void keep(uint32_t d, uint64_t mine) const {
    if (buckets == 0 || d < kHubMinDegree || ballot((mine >> 32) != 0)) return;
    const hub_ptr b = bucket();
    const hub_ptr deg = b + 2 * kHubWays;
    uint32_t way = 0, least = ~0u;
#pragma unroll
    for (uint32_t k = 0; k < kHubWays; ++k) {
      const uint32_t x = hub_load(deg + k);  // a way being written counts as long
      way = x < least ? k : way;
      least = min(x, least);
    }
    way = uniform32(way);
    least = uniform32(least);
    if (least >= d) return;
    uint32_t old = 0;
    if (lane_id() == 0) {
      uint32_t expect = least;
      __hip_atomic_compare_exchange_strong(deg + way, &expect, d | kHubBusy, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      old = expect;
    }
    if (uniform32(old) != least) return;  // another wavefront took the way
    hub_fence();
    // The row may be here by now, or be going into another way.
    bool twin = false;
#pragma unroll
    for (uint32_t k = 0; k < kHubWays; ++k) {
      const uint32_t x = hub_load(deg + k);
      if (k != way) twin |= x == (d | kHubBusy) || (x == d && holds(b, k));
    }
    if (uniform32(twin ? 1u : 0u)) {
      hub_store(deg + way, least);  // nothing of the way was touched
      return;
    }
    hub_store(b + way, kEnd);
    hub_fence();
    hub_store(b + 3 * kHubWays + way * kWave + (uint32_t)lane_id(), (uint32_t)mine);
    hub_store(b + kHubWays + way, want);
    hub_fence();
    hub_store(b + way, cur);
    hub_fence();
    hub_store(deg + way, d);
  }
};

// Empties the cache (the whole workgroup; a barrier follows).
__device__ __forceinline__ void clear_hubs(hub_ptr base, uint32_t buckets) {
  for (uint32_t i = threadIdx.x; i < buckets * kHubBucketWords; i += blockDim.x) {
    const uint32_t k = i % kHubBucketWords;
    base[i] = k < kHubWays ? kEnd : 0u;
  }
}

}  // namespace fw
