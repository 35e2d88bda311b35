// qkv_select.h — device helpers of the rank selections (assign.hip, assign_long.hip, controller.hip): order keys
// and prefix counts over a workgroup of 1024 threads.  Internal to the GPU library.
#pragma once

#include "qkv_common.h"

namespace qkv {

constexpr int kSelectThreads = 1024;
constexpr int kSelectWaves = kSelectThreads / kWaveSize;

// Key that grows as the rank grows: smaller key = better score.  -0 ranks below +0.
__device__ inline uint32_t rank_key(float score) {
  const uint32_t x = __float_as_uint(score);
  const uint32_t up = (x & 0x80000000u) ? ~x : (x | 0x80000000u);   // ascending in the score
  return ~up;
}

__device__ inline uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// Histograms in LDS: additions of several lanes to one word are made one after the other, so scores that crowd together (one
// value, a few, a narrow range) slow a sweep down.  Where the lanes of a wave crowd, those that share the first
// one's bucket are counted and added at once (16384 tokens of one value, first sweep of assign.hip with two copies: 52 -> 42 us
// in all; asked once per wave and not per key, which cost 1 us of 8 where they do not crowd).
//
// Whether they do: at least half of the lanes with a key (on) are in the bucket d of the first of them.
__device__ inline bool lanes_crowd(uint32_t d, bool on) {
  const uint64_t all = __builtin_amdgcn_ballot_w64(on);
  if (all == 0ull) return false;
  const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)__builtin_ctzll(all));
  return 2 * __builtin_popcountll(__builtin_amdgcn_ballot_w64(on && d == first)) >= __builtin_popcountll(all);
}
// hist[d] += weight for every lane with on.
__device__ inline void add_crowded(uint32_t* hist, uint32_t d, bool on, uint32_t lane, uint32_t weight = 1u) {
  const uint64_t all = __builtin_amdgcn_ballot_w64(on);
  if (all == 0ull) return;
  const uint32_t leader = (uint32_t)__builtin_ctzll(all);
  const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)leader);
  const uint64_t same = __builtin_amdgcn_ballot_w64(on && d == first);
  if (lane == leader) atomicAdd(&hist[first], weight * (uint32_t)__builtin_popcountll(same));
  if (on && d != first) atomicAdd(&hist[d], weight);
}

// Prefix over the waves of a workgroup.  tot[0 .. kSelectWaves) are wave totals in LDS (written before the last
// barrier); the result holds, in lanes 0 .. 15 of every wave, the inclusive running sum.  One LDS read and
// four DPP steps: a loop of dependent LDS reads would cost a full LDS latency per wave.
__device__ inline uint32_t scan_wave_totals(const uint32_t* tot, uint32_t lane) {
  uint32_t v = tot[lane & (kSelectWaves - 1u)];
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);    // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);    // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);    // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);    // row_shr:8
  return v;
}
// Sum of the totals of waves [0, w) from that running sum; w must be the same in every lane.
__device__ inline uint32_t waves_below(uint32_t running, uint32_t w) {
  const uint32_t at = uniform(w);
  return at == 0u ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)running, (int)(at - 1u));
}

// Inclusive prefix of N values per thread over the workgroup, thread order, and the totals.  `tot` is LDS scratch that
// the caller does not touch before the next barrier; one barrier inside.
template <int N>
__device__ inline void block_scan(const uint32_t (&v)[N], uint32_t (&inc)[N], uint32_t (&all)[N], uint32_t (*tot)[kSelectWaves],
                                  uint32_t lane, uint32_t wave) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    inc[n] = wave_inclusive_scan(v[n]);
    if (lane == 63) tot[n][wave] = inc[n];
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const uint32_t running = scan_wave_totals(tot[n], lane);
    inc[n] += waves_below(running, wave);
    all[n] = (uint32_t)__builtin_amdgcn_readlane((int)running, kSelectWaves - 1);
  }
}

}  // namespace qkv
