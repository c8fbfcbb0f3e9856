// Node2vec membership in N(prev) over LDS, and evaluator set-up, for the
// walkers that pick with one wavefront or one workgroup.
#pragma once

#include "fw_device.h"
#include "fw_kernels.h"

namespace fw {

extern __shared__ __attribute__((aligned(16))) uint32_t fw_dyn_lds[];

constexpr uint32_t kFib24 = 0x9E3779u;  // 2^24 / golden ratio

// Bucket of key u in a table of 2^(32 - shift) buckets (Fibonacci hashing:
// the top bits of the low word of u times 2^24 / golden ratio).  The 24-bit
// multiply runs at the full VALU rate (a 32-bit one at a quarter); ids from
// 2^24 on hash by their low 24 bits, which costs probes, never exactness.
// (HIP's __umul24 returns a signed int: go through uint32_t.)
__device__ __forceinline__ uint32_t bucket_of(uint32_t u, uint32_t shift) {
  return (uint32_t)__umul24(u, kFib24) >> shift;
}
__device__ __forceinline__ uint32_t log2_ceil(uint64_t x) {
  uint32_t b = 0;
  while ((1ull << b) < x) ++b;
  return b;
}

// u is one of the four cells: the smallest XOR with u is 0.
__device__ __forceinline__ bool has4(uint4 v, uint32_t u) {
  return min(min(v.x ^ u, v.y ^ u), min(v.z ^ u, v.w ^ u)) == 0u;
}

// The bucket has a free cell.  Cells fill in order (an insert takes the first
// free one), so that is the last cell being free.
__device__ __forceinline__ bool open4(uint4 v) { return v.w == kEnd; }

// Membership in N(prev) for one node2vec hop, by a wave-uniform mode:
//   0  binary search of the sorted row in global memory;
//   1  exact hash set in LDS: nb buckets of 4 cells (16 bytes) at
//      fw_dyn_lds[base, base + 4 nb), kEnd marks an empty cell; a key lives
//      in the first bucket, in probe order from its hash, that had a free cell
//      when it was inserted, so a lookup stops at a hit or at a bucket with a
//      free cell.
// (Mode 2, the merge of sorted rows, has its own code: merge_chunk.)
// One type for all modes keeps a single copy of the sampler in the kernel.
struct MemberAny {
  int mode;
  uint32_t base, bmask, shift;
  const uint32_t* __restrict__ adj;
  uint64_t po, pd;

  // base is a multiple of 4 cells, so a bucket is one aligned 16-byte read.
  __device__ __forceinline__ uint4 bucket(uint32_t b) const {
    return reinterpret_cast<const uint4*>(fw_dyn_lds)[(base >> 2) + b];
  }
  __device__ __forceinline__ bool probe_rest(uint32_t u, uint32_t b) const {
    for (;;) {
      b = (b + 1) & bmask;
      const uint4 v = bucket(b);
      if (has4(v, u)) return true;
      if (open4(v)) return false;
    }
  }
  // f[j] = fin if u[j] is in N(prev), else fout.  Choosing the factor inside
  // the lookup keeps the hits in lane masks on the common path; only the
  // rare longer probes update a factor under a lane mask.
  __device__ __forceinline__ void factors4(const uint32_t u[4], uint32_t fin, uint32_t fout,
                                           uint32_t f[4]) const {
    if (mode == 1) {
      uint32_t b[4];
      uint4 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        b[j] = bucket_of(u[j], shift);
        v[j] = bucket(b[j]);
      }
      bool more = false;
      bool done[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool hit = has4(v[j], u[j]);
        f[j] = hit ? fin : fout;
        done[j] = hit | open4(v[j]);
        more |= !done[j];
      }
      if (more) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (!done[j]) f[j] = probe_rest(u[j], b[j]) ? fin : fout;
      }
      return;
    }
    bool hit[4];
    row_contains4(adj, po, pd, u, hit);
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = hit[j] ? fin : fout;
  }
};

// Adds key u to the hash set of MemberAny's mode 1 (any lanes, concurrently).
__device__ __forceinline__ void hash_insert(uint32_t base, uint32_t bmask, uint32_t shift,
                                            uint32_t u) {
  uint32_t b = bucket_of(u, shift);
  for (;;) {
    uint32_t j = 0;
    for (; j < 4; ++j) {
      const uint32_t old = atomicCAS(&fw_dyn_lds[base + 4 * b + j], kEnd, u);
      if (old == kEnd || old == u) break;
    }
    if (j < 4) break;
    b = (b + 1) & bmask;
  }
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A node2vec hop whose N(prev) is more than this many times longer than
// N(cur) looks each of N(cur)'s keys up by binary search of N(prev) in global
// memory (few keys; the top levels of a hub's row stay in cache); a shorter
// N(prev) goes to the hash set or the merge.  Full passes on one MI355X for
// ratios 16, 32, 64 and 128: R-MAT-22 node2vec 1308, 1272, 1275 and
// 1330 ms; Chung-Lu 227M node2vec, 1M queries, 7157, 7084, 7021 and 6992 ms.
// With the hubs' totals kept, ratios 16, 32 and 64: 524,288 walks on R-MAT-22
// 133.8, 128.0 and 128.6 ms, 200,003 unweighted walks of 40 hops on Chung-Lu
// 2^20, whose rows stay in the last-level cache, 17.7, 17.7 and 18.4 ms; ratios
// 32 and 64: the first 1M queries of Chung-Lu 227M 3669 and 3576 ms.  32 is
// within 3 % of the better one on each.
constexpr uint64_t kSearchRatio = 32;

struct Table {
  uint32_t base, cells;   // this wavefront's LDS region
  uint32_t bmask, shift;  // geometry of the hash set
  int kind;               // 0: global search, 1: hash set, 2: merge of sorted rows
  uint64_t po, pd;        // N(prev)
};

// Chooses (and for the hash set builds) the membership structure of N(prev)
// for one node2vec hop from a vertex of degree d, with the wavefront's lanes.
__device__ __forceinline__ void build_table(Table& tb, const uint32_t* __restrict__ adj,
                                            uint64_t d, int lane, bool allow_merge = true) {
  tb.kind = 0;
  if (tb.pd == 0 || tb.pd > kSearchRatio * d) return;
  if (2 * tb.pd > tb.cells) {
    // Too large for the hash set: merge the sorted rows (the region must
    // hold at least one 256-entry staging round).
    if (allow_merge && tb.cells >= 4 * kWave) tb.kind = 2;
    return;
  }
  // The table takes the whole region: a smaller N(prev) gets a lower load,
  // and a lookup then almost never needs a second bucket (with 64 lanes and
  // four lookups each, any lane needing one costs the whole wavefront).
  const uint32_t bits = log2_ceil(tb.cells / 4);  // cells: a power of two >= 64
  tb.bmask = (1u << bits) - 1;
  tb.shift = 32 - bits;
  const uint4 empty = make_uint4(kEnd, kEnd, kEnd, kEnd);
  for (uint32_t i = lane; i < tb.cells / 4; i += kWave)
    reinterpret_cast<uint4*>(fw_dyn_lds + tb.base)[i] = empty;
  wave_sync_lds();
  for (uint64_t i = lane; i < tb.pd; i += kWave) {
    hash_insert(tb.base, tb.bmask, tb.shift, adj[tb.po + i]);
  }
  wave_sync_lds();
  tb.kind = 1;
}

template <int ALGO, bool WEIGHTED, class MEM>
__device__ __forceinline__ Eval<ALGO, WEIGHTED, MEM> base_eval(const DevGraph& g,
                                                              const DevParams& prm, uint64_t o,
                                                              uint32_t prev, uint32_t t) {
  Eval<ALGO, WEIGHTED, MEM> ev;
  ev.adj = g.adj;
  ev.w = g.w;
  ev.lab = g.lab;
  ev.o = o;
  ev.first = (t == 0);
  ev.prev = prev;
  ev.f_ret = prm.f_ret;
  ev.f_in = prm.f_in;
  ev.f_out = prm.f_out;
  ev.want = (ALGO == kMetaPath) ? schema_label(prm, t) : 0u;
  ev.qa = 0;
  ev.narrow = false;
  ev.sum32 = false;
  return ev;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  const int lo = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)v);
  const int hi = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)(v >> 32));
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

}  // namespace fw
