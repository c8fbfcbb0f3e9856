// Group totals of hub rows, kept in LDS for the length of a launch.
//
// Walks meet a vertex in proportion to its degree and a hop's first pass
// streams the whole row, so on power-law graphs a few rows take most of the
// traffic (the 300 longest rows of R-MAT-22 hold 56 % of the entries that
// walks scan, those of Chung-Lu 2^22, gamma 2.1, 93 %).  The first pass of
// an algorithm whose weights depend only on the vertex (and MetaPath's wanted
// label) leaves the same 64 group totals on every visit: the wavefronts of a
// workgroup share them here, and a later visit reads 64 words from LDS and
// one group of the row, 1/64 of it.  Measured on one MI355X, before and after
// (64 totals to a row): 524,288 weighted DeepWalk walks of 80 hops on R-MAT-22
// 48.8 and 35.8 ms, node2vec 142.4 and 137.9 ms (raw weight totals of the rows
// that take the regrouped pass), 1,048,576 PPR walks from its largest hub 24.8
// and 10.4 ms, 2,097,152 MetaPath walks of 20 hops on Chung-Lu 2^22 46.0 and
// 27.3 ms.
//
// Layout: two regions of buckets of four ways, each way a key (vertex, label),
// its degree and totals of 32 bits (rows with a larger total are not kept): 64
// in the first region, which is for the longest rows, and 16, each of four
// groups, in the second, which so holds four times as many rows in the same
// space and reads 1/16 of them on a visit.  A quarter of the space goes to
// the first.  A row replaces the shortest way of its bucket if that is shorter
// than itself, so a way's degree only grows; the top bit of the degree marks a
// way being written.  Readers never wait: they read the key, the totals and
// the key again.  A way that changed in between held another row of strictly
// larger degree meanwhile and cannot have got the old key back.
//
// All ways of 64 totals against this split: the DeepWalk pass above 26.9 and
// 23.1 ms, MetaPath 21.0 and 19.2 ms, node2vec 128.0 and 127.3 ms, PPR 5.6 and
// 5.7 ms (its hub is in either; an eighth or half of the space for the first
// region stays within 3 % on all of them).
#pragma once

#include "fw_device.h"

namespace fw {

// Rows from this degree on are looked up and kept.
constexpr uint32_t kHubMinDegree = 2048;
// Rows from this degree on go to the region of 64 totals, if they find a way.
constexpr uint32_t kHubLongDegree = 32768;
constexpr uint32_t kHubWays = 4;
constexpr uint32_t kHubBusy = 0x80000000u;
constexpr uint32_t kHubFew = 16;  // totals of a way of the second region
// Words of a bucket: keys, labels, degrees, totals.
constexpr uint32_t kHubBucketWords = 3 * kHubWays + kHubWays * kWave;
constexpr uint32_t kHubFewBucketWords = 3 * kHubWays + kHubWays * kHubFew;

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

// Group layout of `len` quads: at most 64 groups of per_group 64-quad chunks.
struct GroupSplit {
  uint32_t gsz, groups;
  __device__ __forceinline__ explicit GroupSplit(uint32_t len) {
    const uint32_t chunks = (len + kWave - 1) / kWave;
    const uint32_t per_group = (chunks + kWave - 1) / kWave;
    gsz = (per_group ? per_group : 1) * kWave;
    groups = (len + gsz - 1) / gsz;
  }
};

// No cache: every first pass streams its row.
struct NoHubs {
  __device__ __forceinline__ bool find(uint32_t, GroupSplit&, uint64_t&) const { return false; }
  __device__ __forceinline__ void keep(uint32_t, uint64_t) const {}
};

// The cache as seen from one hop: its row's key.
struct Hubs {
  hub_ptr base;                    // the first region, then the second
  uint32_t buckets, few_buckets;   // 0: none
  uint32_t cur, want;

  __device__ __forceinline__ uint32_t hash() const {
    return (cur ^ (want * 0x85EBCA6Bu)) * 0x9E3779B1u;
  }
  __device__ __forceinline__ hub_ptr bucket() const {
    return base + __umulhi(hash(), buckets) * kHubBucketWords;
  }
  __device__ __forceinline__ hub_ptr few_bucket() const {
    return base + buckets * kHubBucketWords + __umulhi(hash(), few_buckets) * kHubFewBucketWords;
  }
  __device__ __forceinline__ bool holds(hub_ptr b, uint32_t way) const {
    return hub_load(b + way) == cur && hub_load(b + kHubWays + way) == want;
  }

  // Lane g < n gets total g of the row, if bucket b holds it.
  __device__ __forceinline__ bool find_in(hub_ptr b, uint32_t n, uint64_t& mine) const {
    uint32_t way = kHubWays;
#pragma unroll
    for (uint32_t k = 0; k < kHubWays; ++k) way = holds(b, k) ? k : way;
    way = uniform32(way);
    if (way == kHubWays) return false;
    hub_fence();
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t tot = hub_load(b + 3 * kHubWays + way * n + (lane < n ? lane : 0u));
    hub_fence();
    if (!uniform32(holds(b, way) ? 1u : 0u)) return false;
    mine = lane < n ? tot : 0u;
    return true;
  }

  // Lane g gets the total of group g of the row, if it is here; a row kept
  // with 16 totals has groups four times as long, which sp then says.  (d: the
  // row's degree; every lane of the wavefront calls.)
  __device__ __forceinline__ bool find(uint32_t d, GroupSplit& sp, uint64_t& mine) const {
    if (d < kHubMinDegree) return false;
    if (buckets != 0 && d >= kHubLongDegree && find_in(bucket(), kWave, mine)) return true;
    if (few_buckets == 0 || !find_in(few_bucket(), kHubFew, mine)) return false;
    sp.gsz *= kWave / kHubFew;
    sp.groups = (sp.groups + kWave / kHubFew - 1) / (kWave / kHubFew);
    return true;
  }

  // Offers the row's n totals, in lanes 0, step, 2 step, ...; whether it is
  // there now or is going to be.
  __device__ __forceinline__ bool keep_in(hub_ptr b, uint32_t n, uint32_t step, uint32_t d,
                                          uint32_t total) const {
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
    if (least >= d) return false;
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t old = 0;
    if (lane == 0) {
      uint32_t expect = least;
      __hip_atomic_compare_exchange_strong(deg + way, &expect, d | kHubBusy, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      old = expect;
    }
    if (uniform32(old) != least) return true;  // another wavefront took the way
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
      return true;
    }
    hub_store(b + way, kEnd);
    hub_fence();
    if (lane % step == 0) hub_store(b + 3 * kHubWays + way * n + lane / step, total);
    hub_store(b + kHubWays + way, want);
    hub_fence();
    hub_store(b + way, cur);
    hub_fence();
    hub_store(deg + way, d);
    return true;
  }

  // Offers the row's totals (lane g: group g's).
  __device__ __forceinline__ void keep(uint32_t d, uint64_t mine) const {
    if (d < kHubMinDegree) return;
    if (buckets != 0 && d >= kHubLongDegree && !ballot((mine >> 32) != 0) &&
        keep_in(bucket(), kWave, 1, d, (uint32_t)mine))
      return;
    if (few_buckets == 0) return;
    // Totals of four groups, in every fourth lane.
    uint64_t four = mine + dpp64<0xB1, 0xF>(mine);  // quad_perm 1 0 3 2
    four += dpp64<0x4E, 0xF>(four);                 // quad_perm 2 3 0 1
    if (!ballot((four >> 32) != 0))
      (void)keep_in(few_bucket(), kHubFew, kWave / kHubFew, d, (uint32_t)four);
  }
};

// Buckets of both regions in `words` words of LDS.
inline void hub_buckets_in(size_t words, uint32_t* buckets, uint32_t* few_buckets) {
  *buckets = (uint32_t)(words / 4 / kHubBucketWords);
  *few_buckets = (uint32_t)((words - (size_t)*buckets * kHubBucketWords) / kHubFewBucketWords);
}

// Empties the cache (the whole workgroup; a barrier follows).
__device__ __forceinline__ void clear_hubs(const Hubs& h) {
  const uint32_t first = h.buckets * kHubBucketWords;
  const uint32_t all = first + h.few_buckets * kHubFewBucketWords;
  for (uint32_t i = threadIdx.x; i < all; i += blockDim.x) {
    const uint32_t k = i < first ? i % kHubBucketWords : (i - first) % kHubFewBucketWords;
    h.base[i] = k < kHubWays ? kEnd : 0u;
  }
}

}  // namespace fw
