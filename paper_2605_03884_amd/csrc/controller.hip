// controller.hip — the bit-width controller on the device: the network that scores tokens
// (paper Sec. 4.1.2) and the allocator that follows the budgeted objective of Sec. 3.3
// literally.
//
// Network: 6 features per token -> 64 hidden units (ReLU) -> one score, 512 parameters (no
// output bias: it cannot change a ranking).  One token per thread; the parameters arrive as
// a kernel argument.  fp32 in a fixed order:
// a hidden unit starts at its bias and takes one fused multiply-add per feature in feature
// order; the score starts at +0 and takes one fused multiply-add per hidden unit in unit
// order.
//
// Allocator: every token starts at 2 bits; the upgrades 2->4, 4->8, 8->16 cost 2, 4, 8 bits
// and, with the error model eps(b) = 1 / (2^b - 1), gain S * 2/15, S * 4/255, S * 32/65535
// per bit.  All 3T upgrades are ranked by (gain per bit descending, level ascending, token
// ascending) and the longest prefix that fits the budget is taken.  No sort: a radix select
// over the 32-bit gain keys, with histograms weighted by cost, finds the key at which the
// budget runs out and what is left of the budget there; the upgrades with exactly that key
// are then admitted level by level, by increasing token index, until one does not fit.
#include "qkv_select.h"

namespace qkv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFeatures = 6, kHidden = 64;

// The parameters go through LDS, a hidden unit's eight side by side: read straight from the arguments they are 35
// scalar loads that each wait for the one before (registers hold only four of them at a time), which made
// 8192 tokens take 9.2 us; 5.0 now.  TOKENS per thread: launch_controller.
template <int TOKENS>
__global__ __launch_bounds__(256) void controller_kernel(const float* __restrict__ features, uint32_t T,
                                                         qkv_controller_t p, float* __restrict__ scores) {
  __shared__ __attribute__((aligned(16))) float unit[kHidden][8];       // six weights, bias, output weight
  const uint32_t t0 = blockIdx.x * (256u * TOKENS) + threadIdx.x;
  float x[TOKENS][kFeatures], s[TOKENS];
#pragma unroll
  for (int k = 0; k < TOKENS; ++k) {
    const uint32_t t = t0 + 256u * k;
    s[k] = 0.0f;
#pragma unroll
    for (int i = 0; i < kFeatures; ++i) x[k][i] = 0.0f;
    if (t < T) {
      const float2* row = reinterpret_cast<const float2*>(features + (uint64_t)t * kFeatures);   // 24-byte rows
      const float2 x01 = row[0], x23 = row[1], x45 = row[2];
      x[k][0] = x01.x; x[k][1] = x01.y; x[k][2] = x23.x; x[k][3] = x23.y; x[k][4] = x45.x; x[k][5] = x45.y;
    }
  }
  const float* w1 = &p.w1[0][0];
  for (uint32_t i = threadIdx.x; i < kHidden * kFeatures; i += 256u) unit[i / kFeatures][i % kFeatures] = w1[i];
  if (threadIdx.x < kHidden) unit[threadIdx.x][6] = p.b1[threadIdx.x];
  else if (threadIdx.x < 2u * kHidden) unit[threadIdx.x - kHidden][7] = p.w2[threadIdx.x - kHidden];
  __syncthreads();
#pragma unroll 16 / TOKENS
  for (int j = 0; j < kHidden; ++j) {
    const float4 u0 = *reinterpret_cast<const float4*>(&unit[j][0]), u1 = *reinterpret_cast<const float4*>(&unit[j][4]);
#pragma unroll
    for (int k = 0; k < TOKENS; ++k) {
      float a = u1.z;
      a = __builtin_fmaf(x[k][0], u0.x, a);
      a = __builtin_fmaf(x[k][1], u0.y, a);
      a = __builtin_fmaf(x[k][2], u0.z, a);
      a = __builtin_fmaf(x[k][3], u0.w, a);
      a = __builtin_fmaf(x[k][4], u1.x, a);
      a = __builtin_fmaf(x[k][5], u1.y, a);
      const float h = a > 0.0f ? a : 0.0f;       // NaN -> 0
      s[k] = __builtin_fmaf(h, u1.w, s[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < TOKENS; ++k)
    if (t0 + 256u * k < T) scores[t0 + 256u * k] = s[k];
}

// ---- the greedy allocator -----------------------------------------------------------------------
//
// Up to 32768 tokens one workgroup does it in one launch, a thread owning runs of four neighbouring tokens, the next run 256 tokens
// on, whose scores stay in registers (KPT = 2, 8, 16, 32: a short sequence runs short code).  Three passes over the keys: 12, 10 and 10 bits; every
// thread holds its buckets' sums and a workgroup-wide prefix finds the bucket, and the last pass counts the levels
// apart.  Bound by instruction issue and barriers on one compute unit: of 11.0 us for 8192 tokens the widths took 3.7, with three ranks kept for
// every token.  Now a token's class is the number of floors that its gains reach, ranks are only kept in the one wave in which a level's
// share of the last key ends, and class counts come from ballots; the third pass looks once at a token's three keys.  By events, us, before and
// now: 2048 tokens 5.8 / 5.2, 8192 11.6 / 9.3, 16384 19.6 / 14.5, 32768 36.3 / 25.0; fifty different scores 6.3 / 5.4, 12.5 / 10.1, 20.8 /
// 16.2, 38.2 / 28.4; 50499 and more, whose last launch has the same floors, 39.3 / 34.4 and 43.3 / 35.7.
// The first pass's histogram has four copies: with two, scores that crowd together took longer than before (two copies, four, and
// before, us: a narrow range of 32768 tokens 64 / 47 / 52, normally distributed 52 / 43 / 50, one range of 4096 13.3 / 11.5 /
// 11.5; uniform 8192 11.4 / 11.7 / 16.0); eight cost more to clear and add up (uniform 8192 12.9).  Up to 2048 tokens two do.

constexpr int kThreads = kSelectThreads;
constexpr uint32_t kTop = 4096, kSub = 1024;             // buckets of the first pass, and of the two later ones
constexpr uint32_t kLongFrom = 32768;                    // tokens beyond which several workgroups share the work

__device__ constexpr float kPerBit[3] = {(float)(2.0 / 15.0), (float)(4.0 / 255.0), (float)(32.0 / 65535.0)};

// Key of an upgrade: grows as the gain per bit falls.  The gain is +0 or positive, so its bit
// pattern orders like its value.
__device__ inline uint32_t gain_key(float score, int level) {
  const float s = score > 0.0f ? score : 0.0f;     // negative and NaN scores count as 0
  return ~__float_as_uint(s * kPerBit[level]);
}

// How many of the upgrades with exactly the last key are admitted: level by level until one does not fit; nothing
// after it is taken.  left: units (of 2 bits) still free; the levels cost 1, 2, 4.
__device__ inline void split_last_key(uint32_t left, const uint32_t (&n)[3], uint32_t (&quota)[3], bool& tied) {
  quota[0] = min(n[0], left);
  bool full = quota[0] == n[0];
  left -= quota[0];
  quota[1] = full ? min(n[1], left / 2u) : 0u;
  full = full && quota[1] == n[1];
  left -= 2u * quota[1];
  quota[2] = full ? min(n[2], left / 4u) : 0u;
  tied = false;
#pragma unroll
  for (int l = 0; l < 3; ++l) tied = tied || (quota[l] != 0u && quota[l] != n[l]);
}

// What an upgrade's gain must reach, as bits: taken if its bits are >= floor[level], so a token's class is the number of levels whose floor
// it reaches - a level's gain is at most that of the level before, and a level with a share of the last key has all of the level before it
// admitted.  (A key of 0 does not occur: the largest gain is infinity.)
__device__ inline void gain_floors(uint32_t kstar, const uint32_t (&quota)[3], uint32_t (&floor)[3]) {
#pragma unroll
  for (int l = 0; l < 3; ++l) floor[l] = ~kstar + (quota[l] == 0u ? 1u : 0u);
}

// If a level is admitted in part (tied), it is the last one with a share of the last key: the levels before it are full.
__device__ inline int level_in_part(const uint32_t (&quota)[3]) { return quota[2] != 0u ? 2 : quota[1] != 0u ? 1 : 0; }
__device__ inline float per_bit(int level) { return level == 0 ? kPerBit[0] : level == 1 ? kPerBit[1] : kPerBit[2]; }

template <int KPT>
__global__ __launch_bounds__(kThreads) void greedy_kernel(const float* __restrict__ scores, uint32_t T, uint32_t spare,
                                                          uint8_t* __restrict__ bits, unsigned long long* __restrict__ counts4,
                                                          bool aligned) {
  constexpr uint32_t kCopies = KPT <= 2 ? 2u : 4u;          // of the first pass's histogram, see above
  constexpr int V = KPT < 4 ? KPT : 4, kChunks = KPT / V;   // a thread's tokens: kChunks times V neighbours
  typedef float floats __attribute__((ext_vector_type(V)));
  __shared__ __attribute__((aligned(16))) uint32_t hist[kTop * kCopies];    // first pass: bucket d, copy c at [kCopies d + c]
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ uint32_t sel_digit, sel_left, sel_same[3];
  __shared__ uint32_t class_tot[3];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  // token i of a thread is t0 + at(i), one that exists if at(i) < rest
  const uint32_t wave_t0 = wave * (uint32_t)(kWaveSize * KPT), t0 = wave_t0 + lane * V;
  const int rest = (int)T - (int)t0;
  const auto at = [](int i) { return i / V * kWaveSize * V + i % V; };
  const bool whole = aligned && wave_t0 + (uint32_t)(kWaveSize * KPT) <= T;           // every lane's tokens, vector loads
  float mine[KPT];                                          // the scores, negative ones and NaN as 0
  if (whole) {
    floats f[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) f[c] = *reinterpret_cast<const floats*>(scores + t0 + c * kWaveSize * V);
#pragma unroll
    for (int i = 0; i < KPT; ++i) mine[i] = f[i / V][i % V];
  } else {
#pragma unroll
    for (int i = 0; i < KPT; ++i) mine[i] = at(i) < rest ? scores[t0 + at(i)] : 0.0f;
  }
  // f(key, level) for every upgrade of the own tokens
  const auto for_each_key = [&](auto&& f) {
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      if (at(i) >= rest) continue;
#pragma unroll
      for (int l = 0; l < 3; ++l) f(gain_key(mine[i], l), l);
    }
  };
  if (tid < 3u) class_tot[tid] = 0;
  // `spare` counts units of 2 bits; the upgrades weigh 1, 2, 4.  If all 7T fit, nothing is selected.
  const bool everything = spare >= 7u * T;
  uint32_t kstar = 0, quota[3] = {0, 0, 0}, floor[3] = {0, 0, 0};
  bool tied = false;
  if (!everything) {
    for (uint32_t i = tid; i < kTop * kCopies / 4u; i += kThreads) reinterpret_cast<u32x4*>(hist)[i] = (u32x4)(0u);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KPT; ++i) mine[i] = mine[i] > 0.0f ? mine[i] : 0.0f;
    for_each_key([&](uint32_t key, int l) { atomicAdd(&hist[(key >> 20) * kCopies + (lane & (kCopies - 1u))], 1u << l); });
    __syncthreads();
    uint32_t c[4];
    if constexpr (kCopies == 2u) {
      const u32x4 h0 = reinterpret_cast<const u32x4*>(hist)[2u * tid], h1 = reinterpret_cast<const u32x4*>(hist)[2u * tid + 1u];
      c[0] = h0.x + h0.y; c[1] = h0.z + h0.w; c[2] = h1.x + h1.y; c[3] = h1.z + h1.w;
    } else {
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i) {
        const u32x4 h = reinterpret_cast<const u32x4*>(hist)[4u * tid + i];
        c[i] = h.x + h.y + h.z + h.w;
      }
    }
    uint32_t own[1] = {c[0] + c[1] + c[2] + c[3]}, inc[1], all[1];
    block_scan<1>(own, inc, all, tot, lane, wave);             // every bucket has been read behind its barrier
#pragma unroll
    for (uint32_t i = 0; i < 4u; ++i) hist[i * kSub + tid] = 0u;
    if (inc[0] > spare && inc[0] - own[0] <= spare) {           // exactly one thread: the total, 7T, exceeds spare
      uint32_t left = spare - (inc[0] - own[0]), d = 0;
      if (left >= c[0]) { left -= c[0]; d = 1; if (left >= c[1]) { left -= c[1]; d = 2; if (left >= c[2]) { left -= c[2]; d = 3; } } }
      sel_digit = 4u * tid + d;
      sel_left = left;
    }
    __syncthreads();
    const uint32_t top = uniform(sel_digit), want1 = uniform(sel_left);
    for_each_key([&](uint32_t key, int l) { if ((key >> 20) == top) atomicAdd(&hist[(key >> 10) & (kSub - 1u)], 1u << l); });
    __syncthreads();
    own[0] = hist[tid];
    block_scan<1>(own, inc, all, tot, lane, wave);
    if (inc[0] > want1 && inc[0] - own[0] <= want1) { sel_digit = tid; sel_left = want1 - (inc[0] - own[0]); }
    __syncthreads();
    const uint32_t high = (top << 10) | uniform(sel_digit), want2 = uniform(sel_left);
#pragma unroll
    for (int i = 0; i < KPT; ++i) {                             // few keys are left: one look at a token's three, and no more in most waves
      uint32_t key[3];
      bool any = false;
#pragma unroll
      for (int l = 0; l < 3; ++l) { key[l] = gain_key(mine[i], l); any = any || (key[l] >> 10) == high; }
      if (__builtin_amdgcn_ballot_w64(any && at(i) < rest) == 0ull) continue;
#pragma unroll
      for (int l = 0; l < 3; ++l)
        if ((key[l] >> 10) == high && at(i) < rest) atomicAdd(&hist[(1u + l) * kSub + (key[l] & (kSub - 1u))], 1u);
    }
    __syncthreads();
    const uint32_t n0 = hist[kSub + tid], n1 = hist[2u * kSub + tid], n2 = hist[3u * kSub + tid];
    own[0] = n0 + 2u * n1 + 4u * n2;
    block_scan<1>(own, inc, all, tot, lane, wave);
    if (inc[0] > want2 && inc[0] - own[0] <= want2) {
      sel_digit = tid; sel_left = want2 - (inc[0] - own[0]);
      sel_same[0] = n0; sel_same[1] = n1; sel_same[2] = n2;
    }
    __syncthreads();
    kstar = (high << 10) | uniform(sel_digit);                  // the key at which the budget runs out
    const uint32_t n[3] = {uniform(sel_same[0]), uniform(sel_same[1]), uniform(sel_same[2])};
    split_last_key(uniform(sel_left), n, quota, tied);
    gain_floors(kstar, quota, floor);                           // everything: floors of 0, which every gain reaches
  } else {
    __syncthreads();
  }

  uint32_t reached[3] = {0, 0, 0};                              // the wave's tokens of class >= 1, 2, 3
  const bool word = V == 4 && whole && (reinterpret_cast<uintptr_t>(bits) & 3u) == 0u;
  const auto store = [&](int c, const uint32_t (&cls)[V]) {
    if constexpr (V == 4) {
      if (word) {
        *reinterpret_cast<uint32_t*>(bits + t0 + c * kWaveSize * V) = (2u << cls[0]) | ((2u << cls[1]) << 8) | ((2u << cls[2]) << 16) | ((2u << cls[3]) << 24);
        return;
      }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) if (at(c * V + i) < rest) bits[t0 + at(c * V + i)] = (uint8_t)(2u << cls[i]);
  };
  // Where a level is admitted in part, tokens with the last key are taken in their order: a wave has room for all of its own, for
  // none, or - one wave - for the first of them.
  uint32_t room = 0;
  bool split = false;
  const int part = level_in_part(quota);
  const float part_bit = per_bit(part);
  if (tied) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      n += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(at(i) < rest && __float_as_uint(mine[i] * part_bit) == ~kstar));
    if (lane == 0u) tot[0][wave] = n;
    __syncthreads();
    const uint32_t before = waves_below(scan_wave_totals(tot[0], lane), wave), most = part == 0 ? quota[0] : part == 1 ? quota[1] : quota[2];
    room = most > before ? most - before : 0u;
    split = room != 0u && room < n;
#pragma unroll
    for (int l = 0; l < 3; ++l) if (l == part && room < n) floor[l] = ~kstar + 1u;
  }
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    uint32_t cls[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      cls[i] = 0;
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        const bool taken = __float_as_uint(mine[c * V + i] * kPerBit[l]) >= floor[l];
        cls[i] += taken;
        reached[l] += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(taken && at(c * V + i) < rest));
      }
    }
    if (split) {
      uint32_t rank = 0, n = 0;                                 // the wave's tokens with the last key in front of the thread's
      bool same[V];
#pragma unroll
      for (int i = 0; i < V; ++i) {
        same[i] = at(c * V + i) < rest && __float_as_uint(mine[c * V + i] * part_bit) == ~kstar;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(same[i]);
        rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, rank));
        n += (uint32_t)__builtin_popcountll(mask);
      }
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const bool taken = same[i] && rank < room;
        cls[i] += taken;
        rank += same[i];
        const uint32_t more = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(taken));
#pragma unroll
        for (int l = 0; l < 3; ++l) reached[l] += l == part ? more : 0u;
      }
      room -= min(room, n);
    }
    store(c, cls);
  }
  if (counts4 != nullptr) {
    if (lane < 3u) atomicAdd(&class_tot[lane], lane == 0u ? reached[0] : lane == 1u ? reached[1] : reached[2]);
    __syncthreads();
    if (tid < 4u) counts4[tid] = (tid == 0u ? T : class_tot[tid - 1u]) - (tid == 3u ? 0u : class_tot[tid]);
  }
}

// ---- longer sequences ------------------------------------------------------------------------------
//
// The same three passes as launches with several workgroups sharing the tokens, then one workgroup that settles the last key
// and one launch that writes the widths.  As in assign_long.hip a pass leaves one histogram per workgroup, the next
// pass's workgroups each add them up, and the histograms live in the bits array, which nothing final is written to
// before the last launch; what that launch's workgroups need is left at the start of their own part of it.  A workgroup's
// histograms take 20 KiB, so there is one workgroup per 20 KiB of tokens: a single one up to 41758 tokens, 6 at 128K, 64 - the
// most - from 1.3 M on.  One workgroup re-reading every score in six sweeps, and the chain: 32769 tokens 106 and 40 us, 41000
// 130 and 48, 42000 (two workgroups) 133 and 32, 62000 201 and 40, 128K 452 and 35, 1M 3619 and 58.

constexpr uint32_t kMaxParts = 64;

struct GreedyTail {
  uint32_t prefix[2], left[2];               // after the first and the second pass
  uint32_t below[kMaxParts][3];              // a workgroup's keys in front of the second prefix, by level
};

struct GreedyPart {
  uint32_t kstar, tied, quota[3], same[3];   // same: keys of earlier workgroups that equal kstar
};

struct GreedyArgs {
  const float* scores;
  uint32_t tokens, per, parts, spare, aligned;
  uint8_t* bits;
  uint8_t* hist;                             // `parts` times kPartWords words, then the tail
  unsigned long long* counts4;
};

constexpr uint32_t kPartWords = kTop + kSub;               // the third pass's 3 x 1024 counts take the place of the first one's

__device__ inline uint32_t* part_hist(const GreedyArgs& a, uint32_t b) { return reinterpret_cast<uint32_t*>(a.hist) + (uint64_t)b * kPartWords; }
__device__ inline GreedyTail* tail_of(const GreedyArgs& a) { return reinterpret_cast<GreedyTail*>(part_hist(a, a.parts)); }
__device__ inline GreedyPart* part_of(const GreedyArgs& a, uint32_t b) {
  return reinterpret_cast<GreedyPart*>((reinterpret_cast<uint64_t>(a.bits) + (uint64_t)b * a.per + 15u) & ~(uint64_t)15u);
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void greedy_pass_kernel(GreedyArgs a) {
  constexpr uint32_t kWords = PASS == 0 ? kTop * 2u : PASS == 1 ? kSub : 3u * kSub;
  __shared__ __attribute__((aligned(16))) uint32_t hist[kWords];
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ uint32_t sel_prefix, sel_left;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, b = blockIdx.x;
  const uint32_t t0 = b * a.per, t1 = min(t0 + a.per, a.tokens);
  GreedyTail* tail = tail_of(a);
  for (uint32_t i = tid; i < kWords / 4u; i += kThreads) reinterpret_cast<u32x4*>(hist)[i] = (u32x4)(0u);
  uint32_t prefix = 0;
  if constexpr (PASS > 0) {                                  // the bucket of the pass before, from everybody's histograms
    uint32_t c[4] = {0, 0, 0, 0};
    if constexpr (PASS == 1) {
#pragma unroll 4
      for (uint32_t p = 0; p < a.parts; ++p) {
        const u32x4 h = reinterpret_cast<const u32x4*>(part_hist(a, p))[tid];
        c[0] += h.x; c[1] += h.y; c[2] += h.z; c[3] += h.w;
      }
    } else {
#pragma unroll 4
      for (uint32_t p = 0; p < a.parts; ++p) c[0] += part_hist(a, p)[kTop + tid];
    }
    const uint32_t own[1] = {c[0] + c[1] + c[2] + c[3]};
    uint32_t inc[1], all[1];
    block_scan<1>(own, inc, all, tot, lane, wave);
    const uint32_t want = PASS == 1 ? a.spare : tail->left[0];
    if (inc[0] > want && inc[0] - own[0] <= want) {
      uint32_t left = want - (inc[0] - own[0]), d = 0;
      if (PASS == 1) {
        if (left >= c[0]) { left -= c[0]; d = 1; if (left >= c[1]) { left -= c[1]; d = 2; if (left >= c[2]) { left -= c[2]; d = 3; } } }
        sel_prefix = 4u * tid + d;
      } else {
        sel_prefix = (tail->prefix[0] << 10) | tid;
      }
      sel_left = left;
    }
    __syncthreads();
    prefix = uniform(sel_prefix);
    if (b == 0 && tid == 0) { tail->prefix[PASS - 1] = prefix; tail->left[PASS - 1] = sel_left; }
  } else {
    __syncthreads();
  }
  uint32_t below[3] = {0, 0, 0};
  const auto visit = [&](float score) {
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const uint32_t key = gain_key(score, l);
      if constexpr (PASS == 0) {
        atomicAdd(&hist[(key >> 20) * 2u + (lane & 1u)], 1u << l);
      } else if constexpr (PASS == 1) {
        if ((key >> 20) == prefix) atomicAdd(&hist[(key >> 10) & (kSub - 1u)], 1u << l);
      } else {
        if ((key >> 10) == prefix) atomicAdd(&hist[l * kSub + (key & (kSub - 1u))], 1u);
        below[l] += (uint32_t)((key >> 10) < prefix);
      }
    }
  };
  if (a.aligned) {
    for (uint32_t t = t0 + 4u * tid; t < t1; t += 4u * kThreads) {
      if (t + 4u <= t1) {
        const float4 s = *reinterpret_cast<const float4*>(a.scores + t);
        visit(s.x); visit(s.y); visit(s.z); visit(s.w);
      } else {
        for (uint32_t i = t; i < t1; ++i) visit(a.scores[i]);
      }
    }
  } else {
#pragma unroll 4
    for (uint32_t t = t0 + tid; t < t1; t += kThreads) visit(a.scores[t]);
  }
  __syncthreads();
  uint32_t* mine = part_hist(a, b);
  if constexpr (PASS == 0) {
    const u32x4 h0 = reinterpret_cast<const u32x4*>(hist)[2u * tid], h1 = reinterpret_cast<const u32x4*>(hist)[2u * tid + 1u];
    reinterpret_cast<u32x4*>(mine)[tid] = (u32x4){h0.x + h0.y, h0.z + h0.w, h1.x + h1.y, h1.z + h1.w};
  } else if constexpr (PASS == 1) {
    mine[kTop + tid] = hist[tid];
  } else {
#pragma unroll
    for (uint32_t l = 0; l < 3u; ++l) mine[l * kSub + tid] = hist[l * kSub + tid];
    uint32_t inc[3], all[3];
    block_scan<3>(below, inc, all, tot, lane, wave);
    if (tid < 3) tail->below[b][tid] = tid == 0 ? all[0] : tid == 1 ? all[1] : all[2];
  }
}

// The last key, what of it is admitted, and the class counts.  One workgroup.
__global__ __launch_bounds__(kThreads) void greedy_settle_kernel(GreedyArgs a) {
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ uint32_t sel_digit, sel_left, sel_same[3];
  __shared__ uint32_t in_front[3];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const GreedyTail* tail = tail_of(a);
  if (tid < 3u) in_front[tid] = 0u;
  uint32_t n[3] = {0, 0, 0};
#pragma unroll 4
  for (uint32_t p = 0; p < a.parts; ++p) {
#pragma unroll
    for (int l = 0; l < 3; ++l) n[l] += part_hist(a, p)[l * kSub + tid];
  }
  const uint32_t want = tail->left[1], high = tail->prefix[1];
  uint32_t own[1] = {n[0] + 2u * n[1] + 4u * n[2]}, inc[1], all[1];
  block_scan<1>(own, inc, all, tot, lane, wave);
  if (inc[0] > want && inc[0] - own[0] <= want) {
    sel_digit = tid; sel_left = want - (inc[0] - own[0]);
    sel_same[0] = n[0]; sel_same[1] = n[1]; sel_same[2] = n[2];
  }
  __syncthreads();
  const uint32_t digit = uniform(sel_digit), kstar = (high << 10) | digit;
  const uint32_t same[3] = {uniform(sel_same[0]), uniform(sel_same[1]), uniform(sel_same[2])};
  uint32_t quota[3];
  bool tied;
  split_last_key(uniform(sel_left), same, quota, tied);
  // upgrades of every level in front of the last key
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    uint32_t v = tid < digit ? n[l] : 0u;
    if (tid < a.parts) v += tail->below[tid][l];
    const uint32_t sum = wave_inclusive_scan(v);
    if (lane == 63 && sum) atomicAdd(&in_front[l], sum);
  }
  uint32_t before = 0;                                        // wave = level, lane = workgroup
  if (wave < 3) {
    const uint32_t mine = lane < a.parts ? part_hist(a, lane)[wave * kSub + digit] : 0u;
    before = wave_inclusive_scan(mine) - mine;
  }
  __syncthreads();                                            // everything has been read: the results may go over it
  if (wave < 3 && lane < a.parts) {
    GreedyPart* p = part_of(a, lane);
    p->same[wave] = before;
    p->quota[wave] = wave == 0 ? quota[0] : wave == 1 ? quota[1] : quota[2];
    if (wave == 0) { p->kstar = kstar; p->tied = tied ? 1u : 0u; }
  }
  if (a.counts4 != nullptr && tid == 0) {                     // an upgrade is only taken with those below it
    const uint32_t t4 = in_front[0] + quota[0], t8 = in_front[1] + quota[1], t16 = in_front[2] + quota[2];
    a.counts4[0] = a.tokens - t4; a.counts4[1] = t4 - t8; a.counts4[2] = t8 - t16; a.counts4[3] = t16;
  }
}

// EVERYTHING: the budget covers 16 bits for every token; no launch has gone before.
template <bool EVERYTHING>
__global__ __launch_bounds__(kThreads) void greedy_write_kernel(GreedyArgs a) {
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ GreedyPart part;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, b = blockIdx.x;
  const uint32_t t0 = b * a.per, t1 = min(t0 + a.per, a.tokens);
  uint32_t kstar = 0, floor[3] = {0, 0, 0};
  uint32_t same = 0, most = 0;                                // of the level that is admitted in part: tokens with the last key in earlier workgroups, and how many are taken
  float part_bit = 0.0f;
  bool tied = false;
  if constexpr (!EVERYTHING) {
    if (tid < sizeof(GreedyPart) / 4u) reinterpret_cast<uint32_t*>(&part)[tid] = reinterpret_cast<const uint32_t*>(part_of(a, b))[tid];
    __syncthreads();                                          // read by now: the stores below may go over it
    kstar = uniform(part.kstar);
    tied = uniform(part.tied) != 0u;
    const uint32_t quota[3] = {uniform(part.quota[0]), uniform(part.quota[1]), uniform(part.quota[2])};
    gain_floors(kstar, quota, floor);
    if (tied) {
      const int level = level_in_part(quota);
      same = uniform(part.same[level]);
      most = uniform(part.quota[level]);
      part_bit = per_bit(level);
#pragma unroll
      for (int l = 0; l < 3; ++l) if (l == level) ++floor[l];
    }
  } else if (b == 0 && tid < 4u && a.counts4 != nullptr) {
    a.counts4[tid] = tid == 3u ? a.tokens : 0u;
  }
  for (uint32_t base = t0; base < t1; base += 4u * kThreads) {
    const uint32_t t = base + 4u * tid;
    const uint32_t n = t < t1 ? min(t1 - t, 4u) : 0u;
    float s[4];
    if (!EVERYTHING && a.aligned && n == 4u) {
      const float4 f = *reinterpret_cast<const float4*>(a.scores + t);
      s[0] = f.x; s[1] = f.y; s[2] = f.z; s[3] = f.w;
    } else {
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i) s[i] = !EVERYTHING && i < n ? a.scores[t + i] : 0.0f;
    }
    uint32_t run = 0;
    if (tied) {                                               // tokens with the last key, in their order
      uint32_t eq[1] = {0}, inc[1], all[1];
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i) eq[0] += (uint32_t)(i < n && __float_as_uint((s[i] > 0.0f ? s[i] : 0.0f) * part_bit) == ~kstar);
      block_scan<1>(eq, inc, all, tot, lane, wave);
      run = same + inc[0] - eq[0];
      same += all[0];
      __syncthreads();                                        // the wave totals are written again
    }
    uint32_t widths = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4u; ++i) {
      uint32_t cls = EVERYTHING ? 3u : 0u;
      if constexpr (!EVERYTHING) {
        const float score = s[i] > 0.0f ? s[i] : 0.0f;        // negative and NaN scores count as 0
#pragma unroll
        for (int l = 0; l < 3; ++l) cls += (uint32_t)(__float_as_uint(score * kPerBit[l]) >= floor[l]);
        if (tied && __float_as_uint(score * part_bit) == ~kstar) cls += (uint32_t)(run++ < most);
      }
      widths |= (2u << cls) << (8u * i);
    }
    if (n == 4u && (reinterpret_cast<uintptr_t>(a.bits) & 3u) == 0u) *reinterpret_cast<uint32_t*>(a.bits + t) = widths;
    else for (uint32_t i = 0; i < n; ++i) a.bits[t + i] = (uint8_t)(widths >> (8u * i));
  }
}

hipError_t launch_greedy_long(const float* scores, uint32_t tokens, uint32_t spare_units, uint8_t* bits,
                              unsigned long long* counts4, hipStream_t stream) {
  GreedyArgs a;
  a.scores = scores;
  a.tokens = tokens;
  a.spare = spare_units;
  a.aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0;
  a.bits = bits;
  a.counts4 = counts4;
  // the bits array is all the scratch there is: as many workgroups as their histograms fit into it
  const uint64_t room = (uint64_t)tokens - 15u - sizeof(GreedyTail);
  uint64_t parts = room / (kPartWords * sizeof(uint32_t));
  if (parts > kMaxParts) parts = kMaxParts;
  a.per = (uint32_t)((tokens + parts - 1u) / parts + 3u) & ~3u;
  a.parts = (tokens + a.per - 1u) / a.per;
  a.hist = reinterpret_cast<uint8_t*>((reinterpret_cast<uint64_t>(bits) + 15u) & ~(uint64_t)15u);
  const dim3 grid(a.parts), block(kThreads);
  if (spare_units >= 7ull * tokens) {
    hipLaunchKernelGGL(greedy_write_kernel<true>, grid, block, 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(greedy_pass_kernel<0>, grid, block, 0, stream, a);
  hipLaunchKernelGGL(greedy_pass_kernel<1>, grid, block, 0, stream, a);
  hipLaunchKernelGGL(greedy_pass_kernel<2>, grid, block, 0, stream, a);
  hipLaunchKernelGGL(greedy_settle_kernel, dim3(1), block, 0, stream, a);
  hipLaunchKernelGGL(greedy_write_kernel<false>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_controller(const float* features, uint32_t tokens, const qkv_controller_t& params, float* scores,
                             hipStream_t stream) {
  // Beyond 128K tokens the parameters' trips through LDS are what bounds it: two tokens then share one (1, 2 and 4 tokens a
  // thread: 131072 tokens 5.5 / 5.8 / 7.7 us, 200000 7.1 / 6.5 / 7.9, 1M 19.0 / 14.6 / 14.2; without LDS 5.5, 6.4 and 17.9).
  if (tokens <= 131072u)
    hipLaunchKernelGGL(controller_kernel<1>, dim3((tokens + 255u) / 256u), dim3(256), 0, stream, features, tokens, params, scores);
  else
    hipLaunchKernelGGL(controller_kernel<2>, dim3((tokens + 511u) / 512u), dim3(256), 0, stream, features, tokens, params, scores);
  return hipGetLastError();
}

hipError_t launch_greedy(const float* scores, uint32_t tokens, uint32_t spare_units, uint8_t* bits,
                         unsigned long long* counts4, hipStream_t stream) {
  if (tokens > kLongFrom) return launch_greedy_long(scores, tokens, spare_units, bits, counts4, stream);
  const bool aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0;
  const dim3 grid(1), block(kThreads);
  if (tokens <= 2u * kThreads)
    hipLaunchKernelGGL(greedy_kernel<2>, grid, block, 0, stream, scores, tokens, spare_units, bits, counts4, aligned);
  else if (tokens <= 8u * kThreads)
    hipLaunchKernelGGL(greedy_kernel<8>, grid, block, 0, stream, scores, tokens, spare_units, bits, counts4, aligned);
  else if (tokens <= 16u * kThreads)
    hipLaunchKernelGGL(greedy_kernel<16>, grid, block, 0, stream, scores, tokens, spare_units, bits, counts4, aligned);
  else
    hipLaunchKernelGGL(greedy_kernel<32>, grid, block, 0, stream, scores, tokens, spare_units, bits, counts4, aligned);
  return hipGetLastError();
}

}  // namespace qkv
