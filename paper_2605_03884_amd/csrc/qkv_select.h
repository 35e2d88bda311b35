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
