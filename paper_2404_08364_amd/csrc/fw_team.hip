// Walker of small launches: one workgroup per query.
//
// With fewer queries than the chip has wavefronts, a pass takes as long as
// its longest chain of dependent loads, and a hub row streamed by one
// wavefront is most of it (650 KB at one wavefront's few loads in flight).
// Here wavefront 0 of a workgroup leads a query: it walks short hops alone,
// with the other wavefronts parked at a barrier (they take no issue slots),
// and hands the first pass of a long row, or the hash set of a long N(prev),
// to all of them.  What it does alone is kept short as a chain: the draws of
// 64 hops come from one Philox block per lane, a row's bounds from one load,
// the ids of a row's last level are read along with its weights, so that the
// pick costs no further load, and a short N(prev) goes into its hash set from
// the registers it was read to on the hop before, while the bounds of the
// current row are on their way.
//
// Bound: latency; two dependent loads per short hop, three and four barriers
// per long one.  33 weighted DeepWalk walks of 80 hops on R-MAT-20: 490 us with
// a wavefront per query, 262 us here; 3,001 node2vec walks 2404 and 1571 us.
#include "fw_kernels.h"
#include "fw_member.h"
#include "fw_wave_sampler.h"

namespace fw {

namespace {

constexpr int kMaxWaves = 16;
// N(prev) up to this length is hashed by the leader alone.
constexpr uint32_t kSoloPrev = 256;
// LDS cells of the hash set of N(prev) per thread: up to half as many ids.
constexpr uint32_t kCellsPerThread = 32;

// A long hop, as the leader hands it out.
struct Job {
  uint64_t o, po;
  uint32_t d, pd, prev, t;
  uint32_t mode;         // MemberAny's
  uint32_t build;        // the hash set is still to be built
  uint32_t bmask, shift;
  uint32_t done;         // no hop: the walk has ended
};

// The row of a long hop in groups of 64-quad chunks: up to 64 per wavefront.
struct TeamSplit {
  uint32_t per, gsz, groups;
  __device__ __forceinline__ TeamSplit(uint32_t nq, uint32_t waves) {
    const uint32_t chunks = (nq + kWave - 1) / kWave;
    per = (chunks + kWave * waves - 1) / (kWave * waves);
    gsz = per * kWave;
    groups = (nq + gsz - 1) / gsz;
  }
};

__device__ __forceinline__ uint32_t component(uint4 v, uint32_t j) {
  return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
}

// Totals of the groups wave, wave + waves, ... (several at a time, their
// loads issued together).
template <class E, int K>
__device__ __forceinline__ void team_totals(const E& ev, const QuadSlice& s, const TeamSplit& sp,
                                            uint32_t wave, uint32_t waves, uint64_t* totals) {
  const uint32_t lane = (uint32_t)lane_id();
#pragma unroll 1
  for (uint32_t g0 = wave; g0 < sp.groups; g0 += K * waves) {
    uint64_t acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0;
#pragma unroll 1
    for (uint32_t c = lane; c < sp.gsz; c += kWave) {
      typename E::Loaded v[K];
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = ev.load(min((g0 + k * waves) * sp.gsz + c, s.nq - 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t q = (g0 + k * waves) * sp.gsz + c;
        uint64_t w[4];
        ev.weights(v[k], w);
        if (q == 0 || q + 1 >= s.nq) {  // past the row no entry is inside
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (q >= s.nq || !s.inside(q, j)) w[j] = 0;
        }
        acc[k] += (w[0] + w[1]) + (w[2] + w[3]);
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint64_t tot = ev.sum32 ? wave_sum32((uint32_t)acc[k]) : wave_sum(acc[k]);
      if (lane == 0 && g0 + k * waves < sp.groups) totals[g0 + k * waves] = tot;
    }
  }
}

template <int ALGO, bool WEIGHTED>
__global__ __launch_bounds__(kMaxWaves * kWave) void k_walk_team(
    DevGraph g, DevParams prm, const uint32_t* __restrict__ starts, uint32_t length,
    uint64_t seed, uint64_t qid_base, uint32_t* __restrict__ out, uint32_t* __restrict__ status,
    uint32_t cells, uint32_t narrow, uint32_t sum32) {
  __shared__ Job job;
  // After the hash set: the group totals of a long hop.
  uint64_t* totals = reinterpret_cast<uint64_t*>(fw_dyn_lds + cells);
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t wave = uniform32(threadIdx.x / kWave), waves = blockDim.x / kWave;
  const uint64_t query = blockIdx.x;
  uint32_t cur = uniform32(starts[query]);
  if (cur >= g.nv) {
    if (threadIdx.x == 0) flag_bad_start(status);
    return;
  }
  uint32_t* __restrict__ row = out + query * ((uint64_t)length + 1);
  if (threadIdx.x == 0) row[0] = cur;
  if (length == 0) return;

  // The leader's state: the hop's row [o, o + d), the one before [po, po + pd)
  // and, if that was short, its ids (lane i: quad i).
  uint64_t o = 0, po = 0, draws = 0, stops = 0;
  uint32_t d = 0, pd = 0, prev = kEnd, t = 0;
  uint4 ids = make_uint4(0, 0, 0, 0);
  bool have_ids = false, pending = false;
  uint32_t mode = 0, bmask = 0, shift = 0;

  auto evaluator = [&](uint64_t row_o, uint32_t p, uint32_t hop, uint64_t p_o, uint32_t p_d,
                       uint32_t m, uint32_t mask, uint32_t sh) {
    auto ev = base_eval<ALGO, WEIGHTED, MemberAny>(g, prm, row_o, p, hop);
    ev.narrow = narrow != 0;
    ev.sum32 = sum32 != 0;
    ev.mem.mode = (int)m;
    ev.mem.base = 0;
    ev.mem.bmask = mask;
    ev.mem.shift = sh;
    ev.mem.adj = g.adj;
    ev.mem.po = p_o;
    ev.mem.pd = p_d;
    ev.qa = row_o & ~3ull;
    return ev;
  };

  for (;;) {
    if (wave == 0) {
      bool done = false;
      for (;;) {  // hops the leader finishes alone, and the end of a long one
        uint32_t lo = 0, len;
        uint64_t r = 0;
        bool none = false;  // no neighbour to go to
        if (!pending) {
          const uint64_t bound = g.off[(uint64_t)cur + (lane & 1)];
          if (t % kWave == 0) {
            uint64_t word1;
            draws = philox_draw2(seed, qid_base + query, (uint64_t)t + lane, word1);
            if (ALGO == kPPR)
              stops = ballot(__umul64hi(word1, (uint64_t)prm.stop_den) < (uint64_t)prm.stop_num);
          }
          mode = 0;
          if (ALGO == kNode2Vec && t > 0) {
            const QuadSlice ps(o, d);
            po = o;
            pd = d;
            if (pd <= kSoloPrev) {
              mode = 1;
              const uint32_t bits = max(4u, log2_ceil(pd));
              bmask = (1u << bits) - 1;
              shift = 32 - bits;
              const uint4 empty = make_uint4(kEnd, kEnd, kEnd, kEnd);
              for (uint32_t i = lane; i <= bmask; i += kWave)
                reinterpret_cast<uint4*>(fw_dyn_lds)[i] = empty;
              wave_sync_lds();
              if (have_ids) {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j)
                  if (lane < ps.nq && ps.inside(lane, (int)j))
                    hash_insert(0, bmask, shift, component(ids, j));
              } else {
                for (uint32_t i = lane; i < pd; i += kWave)
                  hash_insert(0, bmask, shift, g.adj[po + i]);
              }
              wave_sync_lds();
            }
          }
          o = readlane64(bound, 0);
          d = (uint32_t)(readlane64(bound, 1) - o);
          have_ids = false;
          if (ALGO == kPPR && ((stops >> (t % kWave)) & 1u)) d = 0;
          none = d == 0;
          const QuadSlice s(o, d);
          len = s.nq;
          const bool hash = ALGO == kNode2Vec && t > 0 && mode == 0 && 2 * pd <= cells;
          if (!none && (len > (uint32_t)kWave || hash)) {
            if (hash) {
              mode = 1;
              const uint32_t bits = min(log2_ceil(pd), log2_ceil(cells / 4));
              bmask = (1u << bits) - 1;
              shift = 32 - bits;
            }
            if (lane == 0) {
              job.o = o;
              job.d = d;
              job.po = po;
              job.pd = pd;
              job.prev = prev;
              job.t = t;
              job.mode = mode;
              job.build = hash ? 1u : 0u;
              job.bmask = bmask;
              job.shift = shift;
            }
            pending = true;
            break;
          }
        } else {
          // The groups' totals are in LDS: T, the draw, the group.
          pending = false;
          const QuadSlice s(o, d);
          const TeamSplit sp(s.nq, waves);
          const uint32_t m = (sp.groups + kWave - 1) / kWave;
          uint64_t own = 0;
          for (uint32_t i = 0; i < m; ++i)
            if (lane * m + i < sp.groups) own += totals[lane * m + i];
          const uint64_t incl = wave_incl_scan(own);
          const uint64_t total = readlane64(incl, kWave - 1);
          len = 0;
          none = total == 0;
          if (!none) {
            r = scale_draw(readlane64(draws, (int)(t % kWave)), total);
            const int at = first_lane(ballot(incl > r));
            r -= readlane64(incl - own, at);
            const uint32_t g0 = (uint32_t)at * m;
            const uint64_t x = lane < m && g0 + lane < sp.groups ? totals[g0 + lane] : 0;
            const uint64_t incl2 = wave_incl_scan(x);
            const int at2 = first_lane(ballot(incl2 > r));
            r -= readlane64(incl2 - x, at2);
            lo = (g0 + (uint32_t)at2) * sp.gsz;
            len = min(sp.gsz, s.nq - lo);
          }
        }
        uint32_t next = kEnd;
        if (!none) {
          const QuadSlice s(o, d);
          const auto ev = evaluator(o, prev, t, po, pd, mode, bmask, shift);
          const bool have_r = len != s.nq;  // else the whole row is the last level
          while (len > (uint32_t)kWave) {   // groups of the longest rows
            const GroupSplit sp(len);
            const uint64_t mine = wave_group_totals(ev, s, lo, len, sp);
            const uint64_t incl = wave_incl_scan(mine);
            const int at = first_lane(ballot(incl > r));
            r -= readlane64(incl - mine, at);
            lo += (uint32_t)at * sp.gsz;
            len = min(sp.gsz, len - (uint32_t)at * sp.gsz);
          }
          uint64_t w[4] = {0, 0, 0, 0};
          const uint32_t q = min(lo + lane, s.nq - 1);
          const typename std::remove_const<decltype(ev)>::type::Loaded v = ev.load(q);
          ids = ev.quad_ids(q);
          if (lane < len) {
            ev.weights(v, w);
            if (q == 0 || q + 1 == s.nq) {
#pragma unroll
              for (int j = 0; j < 4; ++j)
                if (!s.inside(q, j)) w[j] = 0;
            }
          }
          const uint64_t u = readlane64(draws, (int)(t % kWave));
          const int64_t idx = pick_in_quads(w, s, lo, len, r, have_r, u, ev.sum32);
          if (idx >= 0) {
            const uint32_t e = (uint32_t)idx + s.lead;
            next = readlane32(component(ids, e & 3u), (int)(e / 4 - lo));
            have_ids = s.nq <= (uint32_t)kWave;
          }
        }
        if (next == kEnd) {
          for (uint64_t p = (uint64_t)t + 1 + lane; p <= length; p += kWave) row[p] = kEnd;
          done = true;
          break;
        }
        prev = cur;
        cur = next;
        ++t;
        if (lane == 0) row[t] = cur;
        if (t == length) {
          done = true;
          break;
        }
      }
      if (lane == 0) job.done = done ? 1u : 0u;
    }
    __syncthreads();
    if (job.done) break;
    // A long hop, all wavefronts.
    const uint64_t j_o = uniform64(job.o), j_po = uniform64(job.po);
    const uint32_t j_d = uniform32(job.d), j_pd = uniform32(job.pd);
    const uint32_t j_mask = uniform32(job.bmask), j_shift = uniform32(job.shift);
    if (ALGO == kNode2Vec && job.build) {
      const uint4 empty = make_uint4(kEnd, kEnd, kEnd, kEnd);
      for (uint32_t i = threadIdx.x; i <= j_mask; i += blockDim.x)
        reinterpret_cast<uint4*>(fw_dyn_lds)[i] = empty;
      __syncthreads();
      for (uint32_t i = threadIdx.x; i < j_pd; i += blockDim.x)
        hash_insert(0, j_mask, j_shift, g.adj[j_po + i]);
      __syncthreads();
    }
    const QuadSlice s(j_o, j_d);
    const auto ev = evaluator(j_o, uniform32(job.prev), uniform32(job.t), j_po, j_pd,
                              uniform32(job.mode), j_mask, j_shift);
    constexpr int kTogether = ALGO == kNode2Vec ? 2 : 4;
    team_totals<typename std::remove_const<decltype(ev)>::type, kTogether>(
        ev, s, TeamSplit(s.nq, waves), wave, waves, totals);
    __syncthreads();
  }
}

template <int ALGO, bool WEIGHTED>
hipError_t go(const LaunchArgs& a, unsigned block, hipStream_t stream) {
  const uint32_t cells = ALGO == kNode2Vec ? kCellsPerThread * block : 0;
  hipLaunchKernelGGL((k_walk_team<ALGO, WEIGHTED>), dim3((unsigned)a.n), dim3(block),
                     cells * sizeof(uint32_t) + block * sizeof(uint64_t), stream, a.g, a.prm, a.starts, a.length, a.seed,
                     a.qid_base, a.out, a.status, cells, a.cfg.narrow, a.cfg.sum32);
  return hipGetLastError();
}

}  // namespace

// Queries per CU up to which a launch takes a workgroup per query.  Times of
// 40 hops here and with a wavefront per query (both forced), us:
//   R-MAT-20 (longest row 64 k), node2vec: 512 queries 322 and 945, 1,024 473
//     and 1071, 2,048 850 and 1116, 3,072 899 and 1180, 4,096 1002 and 1209,
//     6,144 1433 and 1365; weighted DeepWalk: 512 173 and 236, 1,024 178 and
//     235, 2,048 219 and 246, 3,072 251 and 246, 4,096 258 and 256, 6,144 365
//     and 296; PPR: 1,024 85 and 100, 3,072 129 and 143, 6,144 159 and 167;
//   Chung-Lu 2^18 (43 k), node2vec without weights: 512 279 and 514, 1,024 345
//     and 564, 2,048 523 and 637, 3,072 743 and 669, 4,096 808 and 682;
//     weighted DeepWalk: 1,024 166 and 207, 2,048 212 and 247, 3,072 257 and
//     246, 4,096 327 and 263; MetaPath: 512 129 and 166, 1,024 139 and 164,
//     2,048 206 and 180;
//   R-MAT-14 (no row past 3,700), node2vec: 512 203 and 274, 768 224 and 286,
//     1,024 225 and 288, 2,048 287 and 309, 3,072 411 and 327; weighted
//     DeepWalk: 256 118 and 115, 1,024 136 and 118.
// So on graphs with long rows both meet near twelve queries per CU (MetaPath:
// between four and eight), a little earlier or later with the graph; without
// them only node2vec gains, from the hash sets built ahead, clearly up to about
// four.  Degrees between 3,700 and 43,000 were not timed.  A node2vec launch
// here takes most of the LDS of the CUs it runs on and up to half of their
// wavefronts, so launches on several streams overlap less: 256 queries each on
// one, two and four streams, R-MAT-20 node2vec 270, 492 and 961 here against
// 902, 959 and 1931, weighted DeepWalk 135, 251 and 462 against 227, 226 and
// 253; R-MAT-14 node2vec 177, 334 and 643 against 264, 302 and 358.
bool team_walks(const LaunchArgs& a) {
  const bool long_rows = a.max_deg > 8192;
  uint64_t per_cu = 0;
  switch (a.algo) {
    case kNode2Vec: per_cu = long_rows ? 12 : 3; break;
    case kMetaPath: per_cu = long_rows ? 4 : 0; break;
    case kDeepWalk:
    case kPPR: per_cu = long_rows && a.g.w != nullptr ? 12 : 0; break;
    default: break;
  }
  return a.n <= per_cu * (uint64_t)a.num_cus;
}

hipError_t launch_team(const LaunchArgs& a, hipStream_t stream) {
  // As many wavefronts per query as keep about sixteen on every CU.
  const uint64_t cus = (uint64_t)a.num_cus;
  const unsigned block = a.n <= cus ? 1024 : a.n <= 2 * cus ? 512 : a.n <= 4 * cus ? 256 : 128;
  const bool wt = a.g.w != nullptr;
  switch (a.algo) {
    case kDeepWalk: return go<kDeepWalk, true>(a, block, stream);
    case kNode2Vec:
      return wt ? go<kNode2Vec, true>(a, block, stream) : go<kNode2Vec, false>(a, block, stream);
    case kMetaPath:
      return wt ? go<kMetaPath, true>(a, block, stream) : go<kMetaPath, false>(a, block, stream);
    case kPPR: return go<kPPR, true>(a, block, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fw
