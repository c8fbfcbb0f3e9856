// The two parallel reservoir samplers of section 4 for one wavefront (see
// fw_reservoir.hip for the definition of the per-entry words and of the
// visiting orders).  E provides operator()(i): the weight of entry i of the
// sequence.
#pragma once

#include "fw_device.h"

namespace fw {

// Weights and words of quad q (relative entries 4q .. 4q + 3; 0 past d).
template <class E>
__device__ __forceinline__ void quad_entries(const E& ev, uint64_t d, uint64_t q, uint64_t seed,
                                             uint64_t qid, uint32_t t, uint64_t w[4],
                                             uint64_t u[4], bool draw) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t i = 4 * q + j;
    w[j] = i < d ? ev(i) : 0ull;
  }
  if (draw) philox4x64_10(qid, t, q, 1, seed, u);
}

// Last selection among the four entries of a quad, given the running total
// before it; updates the running total.  Returns -1 when none is selected.
__device__ __forceinline__ int64_t quad_select(const uint64_t w[4], const uint64_t u[4],
                                               uint64_t q, uint64_t& running) {
  int64_t sel = -1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    running += w[j];
    if (w[j] != 0 && __umul64hi(u[j], running) < w[j]) sel = (int64_t)(4 * q + j);
  }
  return sel;
}

// The selection of the highest lane that holds one (every lane calls it).
__device__ __forceinline__ int64_t last_selection(int64_t sel) {
  const uint64_t m = ballot(sel >= 0);
  if (!m) return -1;
  const int src = 63 - __builtin_clzll(m);
  return (int64_t)readlane64((uint64_t)sel, src);
}

template <class E>
__device__ __forceinline__ int64_t dprs_pick(const E& ev, uint64_t d, uint64_t seed,
                                             uint64_t qid, uint32_t t) {
  const int lane = lane_id();
  const uint64_t quads = (d + 3) / 4;
  uint64_t base = 0;  // total of the chunks before
  int64_t pick = -1;
  for (uint64_t c = 0; c * kWave < quads; ++c) {
    const uint64_t q = c * kWave + lane;
    uint64_t w[4] = {0, 0, 0, 0}, u[4] = {0, 0, 0, 0};
    if (q < quads) quad_entries(ev, d, q, seed, qid, t, w, u, true);
    const uint64_t s = (w[0] + w[1]) + (w[2] + w[3]);
    const uint64_t incl = wave_incl_scan(s);
    uint64_t running = base + incl - s;
    const int64_t sel = last_selection(quad_select(w, u, q, running));
    if (sel >= 0) pick = sel;
    base += readlane64(incl, kWave - 1);
  }
  return pick;
}

// The same pick as dprs_pick for a row in memory: the pick is the last
// selection, so after a first pass for the total T the chunks are visited from
// the last one, each with the running total that stands before it, and the
// visit ends at the first chunk that selects.  On average half of the row's
// Philox blocks are never drawn; they are most of what a chunk costs.  50,021
// DeepWalk walks of 20 hops on R-MAT-20: 4.49 ms visiting forwards with queries
// assigned statically, 1.94 ms so with queries handed out dynamically and the
// leaner Philox block.  B provides load(q) and weights(v, q, w): the weights
// (B::Weight) of relative quad q (0 past the row), read in two steps, and
// total(quads).
template <class B>
__device__ __forceinline__ int64_t dprs_pick_back(const B& row, uint32_t d, uint64_t seed,
                                                  uint64_t qid, uint32_t t) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t quads = (d + 3) / 4;
  uint64_t end = row.total(quads);  // total of the chunks up to the current one
  if (end == 0) return -1;
  const bool small = (end >> 32) == 0;
  uint32_t c = (quads - 1) / kWave * kWave;
  typename B::Loaded v = row.load(c + lane);
  for (;;) {
    const typename B::Loaded cur = v;
    if (c != 0) v = row.load(c - kWave + lane);  // the next chunk is on its way
    const uint32_t q = c + lane;
    typename B::Weight w[4];
    row.weights(cur, q, w);
    int64_t sel = -1;
    uint64_t chunk;
    if (small) {
      const uint32_t s = (uint32_t)((w[0] + w[1]) + (w[2] + w[3]));
      const uint32_t incl = wave_incl_scan32(s);
      chunk = readlane32(incl, kWave - 1);
      if (chunk != 0) {
        uint64_t u[4];
        philox4x64_10(qid, t, q, 1, seed, u);
        uint32_t running = (uint32_t)(end - chunk) + incl - s;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          running += (uint32_t)w[j];
          // floor(u * running / 2^64) for a 32-bit running total.
          const uint64_t m = (u[j] >> 32) * running + (((uint64_t)(uint32_t)u[j] * running) >> 32);
          if (w[j] != 0 && (uint32_t)(m >> 32) < (uint32_t)w[j]) sel = (int64_t)(4 * q + j);
        }
      }
    } else {
      const uint64_t s = ((uint64_t)w[0] + w[1]) + ((uint64_t)w[2] + w[3]);
      const uint64_t incl = wave_incl_scan(s);
      chunk = readlane64(incl, kWave - 1);
      if (chunk != 0) {
        uint64_t u[4];
        philox4x64_10(qid, t, q, 1, seed, u);
        uint64_t running = end - chunk + incl - s;
        const uint64_t w64[4] = {w[0], w[1], w[2], w[3]};
        sel = quad_select(w64, u, q, running);
      }
    }
    const int64_t pick = last_selection(sel);
    // The first entry of positive weight selects itself, so chunk 0 ends it.
    if (pick >= 0 || c == 0) return pick;
    end -= chunk;
    c -= kWave;
  }
}

template <class E>
__device__ __forceinline__ int64_t zprs_pick(const E& ev, uint64_t d, uint64_t seed,
                                             uint64_t qid, uint32_t t) {
  const int lane = lane_id();
  const uint64_t quads = (d + 3) / 4;
  uint64_t mine = 0;
  for (uint64_t q = lane; q < quads; q += kWave) {
    uint64_t w[4], u[4];
    quad_entries(ev, d, q, seed, qid, t, w, u, false);
    mine += (w[0] + w[1]) + (w[2] + w[3]);
  }
  uint64_t running = wave_incl_scan(mine) - mine;
  int64_t sel = -1;
  for (uint64_t q = lane; q < quads; q += kWave) {
    uint64_t w[4], u[4];
    quad_entries(ev, d, q, seed, qid, t, w, u, true);
    const int64_t s = quad_select(w, u, q, running);
    if (s >= 0) sel = s;
  }
  return last_selection(sel);
}


// zprs_pick for a row in memory (B as above).
template <class B>
__device__ __forceinline__ int64_t zprs_pick_row(const B& row, uint32_t d, uint64_t seed,
                                                 uint64_t qid, uint32_t t) {
  const uint32_t quads = (d + 3) / 4;
  uint64_t mine = 0;
  for (uint32_t q = (uint32_t)lane_id(); q < quads; q += kWave) {
    typename B::Weight w[4];
    row.weights(row.load(q), q, w);
    mine += ((uint64_t)w[0] + w[1]) + ((uint64_t)w[2] + w[3]);
  }
  uint64_t running = wave_incl_scan(mine) - mine;
  int64_t sel = -1;
  for (uint32_t q = (uint32_t)lane_id(); q < quads; q += kWave) {
    typename B::Weight x[4];
    row.weights(row.load(q), q, x);
    const uint64_t w[4] = {x[0], x[1], x[2], x[3]};
    uint64_t u[4];
    philox4x64_10(qid, t, q, 1, seed, u);
    const int64_t s = quad_select(w, u, q, running);
    if (s >= 0) sel = s;
  }
  return last_selection(sel);
}

}  // namespace fw
