// assign_long.hip — the rank-quantile allocator (paper Sec. 3.3), alone or together with the card's planning
// (Sec. 4.2.1), for sequences longer than one workgroup's registers hold.  Same rule and same results as assign.hip.
//
// Five launches on the caller's stream: three histogram passes over the 32-bit order keys (12, 10 and 10 bits), one
// workgroup that settles the cuts, and the pass that writes widths (and tables).  Several workgroups share the
// tokens, each a run of `per` consecutive ones: widths alone one per 14 KiB of tokens, which is what a workgroup's histograms
// take of the bits array (2 at 32769 tokens, 9 at 128K, 64 - the most - from 0.9 M on), with planning one per 8192 (3 at 16385,
// 16 at 128K, 64 from 512K on).  A pass leaves one histogram per workgroup; the next pass's
// workgroups each add all of them up again and find the buckets of the three cuts by themselves, so nothing is
// zeroed beforehand, there are no atomics on global memory and no workgroup waits for another.
//
// What bounds it: five launches' latencies and the few microseconds each needs for its loads to come back.  The
// single workgroup that did this before re-read every score from cache in six sweeps: 446 us for 128K tokens, and 30 us
// for the classification behind it; the chain takes 39 us (5 + 7 + 8 + 9 + 10, kernel trace).  Widths alone: 32769 tokens
// 106 -> 28 us, 62000 204 -> 28, 128K 449 -> 30, 1M 3624 -> 65.
//
// Scratch without a workspace argument: the histograms live where the results go - in the bits array, or, when a
// card is planned, in its slot and order tables - because nothing is final there before the last launch.  The last
// launch must not read what a neighbour overwrites, so the settling workgroup leaves each workgroup's numbers at
// the start of that workgroup's own part of the result, where only it reads and writes.
#include "qkv_plan.h"
#include "qkv_select.h"

namespace qkv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = kSelectThreads;
constexpr uint32_t kMaxParts = 64;           // workgroups: the settling one handles them as the lanes of a wave
constexpr uint32_t kTop = 4096, kSub = 1024; // buckets of the first pass, and of the two later ones for each cut
constexpr int kTopCopies = 4;                // of the first histogram: real scores share sign and exponent

// Numbers between the launches, behind the histograms.
struct Tail {
  uint32_t prefix[2][3];                     // key bits of every cut after the first and the second pass
  uint32_t left[2][3];                       // rank still to descend there
  uint32_t below[kMaxParts][3];              // a workgroup's keys in front of the second prefix
};

// What the last launch's workgroup needs to know, at the start of its own part of the result.
struct Part {
  uint32_t key[3];                           // the key at every cut
  uint32_t quota[3];                         // tokens with exactly that key that still lie in front of the cut
  uint32_t same[3];                          // tokens of earlier workgroups with exactly that key
  uint32_t ahead[3];                         // tokens of earlier workgroups in front of the cut
  uint32_t tied;                             // some cut splits the tokens that share its key
};

struct LongArgs {
  const float* scores;
  uint32_t tokens, per, parts;
  uint32_t cut[3];
  uint32_t aligned;                          // scores on 16 bytes
  uint8_t* hist;                             // `parts` histograms of part_bytes<CNT>(), then the Tail
  uint8_t* result;                           // workgroup b's Part lies at result + b * result_step, rounded up to 16 bytes
  uint64_t result_step;
};

template <typename CNT> constexpr uint32_t part_bytes() { return (kTop + 3u * kSub) * (uint32_t)sizeof(CNT); }

template <typename CNT> __device__ inline Tail* tail_of(const LongArgs& a) {
  return reinterpret_cast<Tail*>(a.hist + (uint64_t)a.parts * part_bytes<CNT>());
}
// Histograms of workgroup b.  The third pass's take the place of the first one's, which nobody reads any more then.
template <typename CNT> __device__ inline CNT* top_hist(const LongArgs& a, uint32_t b) {
  return reinterpret_cast<CNT*>(a.hist + (uint64_t)b * part_bytes<CNT>());
}
template <typename CNT> __device__ inline CNT* mid_hist(const LongArgs& a, uint32_t b) { return top_hist<CNT>(a, b) + kTop; }
template <typename CNT> __device__ inline CNT* low_hist(const LongArgs& a, uint32_t b) { return top_hist<CNT>(a, b); }

__host__ __device__ inline uint64_t part_offset(const uint8_t* result, uint64_t step, uint32_t b) {
  const uint64_t at = reinterpret_cast<uint64_t>(result) + step * b;
  return ((at + 15u) & ~(uint64_t)15u) - reinterpret_cast<uint64_t>(result);
}

// Calls f(key) for every token of [t0, t1), any order; t0 is a multiple of 4.
template <typename F>
__device__ inline void for_each_key(const LongArgs& a, uint32_t t0, uint32_t t1, F&& f) {
  if (a.aligned) {
#pragma unroll 2
    for (uint32_t t = t0 + 4u * threadIdx.x; t < t1; t += 4u * kThreads) {
      if (t + 4u <= t1) {
        const float4 s = *reinterpret_cast<const float4*>(a.scores + t);
        f(rank_key(s.x)); f(rank_key(s.y)); f(rank_key(s.z)); f(rank_key(s.w));
      } else {
        for (uint32_t i = t; i < t1; ++i) f(rank_key(a.scores[i]));
      }
    }
  } else {
#pragma unroll 4
    for (uint32_t t = t0 + threadIdx.x; t < t1; t += kThreads) f(rank_key(a.scores[t]));
  }
}

// One histogram pass (0, 1, 2) over the workgroup's tokens.
template <int PASS, typename CNT>
__global__ __launch_bounds__(kThreads) void long_pass_kernel(LongArgs a) {
  constexpr uint32_t kWords = PASS == 0 ? kTop * kTopCopies : 3u * kSub;
  __shared__ __attribute__((aligned(16))) uint32_t hist[kWords];
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ uint32_t sel_prefix[3], sel_left[3];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, b = blockIdx.x;
  const uint32_t t0 = b * a.per, t1 = min(t0 + a.per, a.tokens);
  Tail* tail = tail_of<CNT>(a);
  const bool live[3] = {a.cut[0] < a.tokens, a.cut[1] < a.tokens, a.cut[2] < a.tokens};
  for (uint32_t i = tid; i < kWords / 4u; i += kThreads) reinterpret_cast<u32x4*>(hist)[i] = (u32x4)(0u);

  if constexpr (PASS == 0) {
    __syncthreads();
    for_each_key(a, t0, t1, [&](uint32_t key) { atomicAdd(&hist[(key >> 20) * kTopCopies + (lane & (kTopCopies - 1u))], 1u); });
    __syncthreads();
    uint32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 h = reinterpret_cast<const u32x4*>(hist)[4u * tid + i];
      c[i] = h.x + h.y + h.z + h.w;
    }
    CNT* dst = top_hist<CNT>(a, b) + 4u * tid;
    if constexpr (sizeof(CNT) == 2) *reinterpret_cast<u32x2*>(dst) = (u32x2){c[0] | (c[1] << 16), c[2] | (c[3] << 16)};
    else *reinterpret_cast<u32x4*>(dst) = (u32x4){c[0], c[1], c[2], c[3]};
  } else {
    // ---- the buckets of the pass before, from everybody's histograms
    uint32_t prefix[3], below[3] = {0, 0, 0};
    if constexpr (PASS == 1) {
      uint32_t c[4] = {0, 0, 0, 0};
#pragma unroll 8
      for (uint32_t p = 0; p < a.parts; ++p) {
        const CNT* src = top_hist<CNT>(a, p) + 4u * tid;
        if constexpr (sizeof(CNT) == 2) {
          const u32x2 h = *reinterpret_cast<const u32x2*>(src);
          c[0] += h.x & 0xFFFFu; c[1] += h.x >> 16; c[2] += h.y & 0xFFFFu; c[3] += h.y >> 16;
        } else {
          const u32x4 h = *reinterpret_cast<const u32x4*>(src);
          c[0] += h.x; c[1] += h.y; c[2] += h.z; c[3] += h.w;
        }
      }
      const uint32_t own[1] = {c[0] + c[1] + c[2] + c[3]};
      uint32_t inc[1], all[1];
      block_scan<1>(own, inc, all, tot, lane, wave);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        uint32_t left = a.cut[k] - (inc[0] - own[0]);
        if (live[k] && inc[0] > a.cut[k] && inc[0] - own[0] <= a.cut[k]) {          // exactly one thread
          uint32_t d = 0;
          if (left >= c[0]) { left -= c[0]; d = 1; if (left >= c[1]) { left -= c[1]; d = 2; if (left >= c[2]) { left -= c[2]; d = 3; } } }
          sel_prefix[k] = 4u * tid + d;
          sel_left[k] = left;
        }
      }
    } else {
      uint32_t own[3] = {0, 0, 0}, inc[3], all[3];
#pragma unroll 4
      for (uint32_t p = 0; p < a.parts; ++p) {
        const CNT* src = mid_hist<CNT>(a, p) + tid;
#pragma unroll
        for (int k = 0; k < 3; ++k) own[k] += src[k * kSub];
      }
      block_scan<3>(own, inc, all, tot, lane, wave);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint32_t want = tail->left[0][k];
        if (live[k] && inc[k] > want && inc[k] - own[k] <= want) {
          sel_prefix[k] = (tail->prefix[0][k] << 10) | tid;
          sel_left[k] = want - (inc[k] - own[k]);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) prefix[k] = live[k] ? uniform(sel_prefix[k]) : 0xFFFFFFFFu;      // no key has that prefix
    if (b == 0 && tid < 3 && (tid == 0 ? live[0] : tid == 1 ? live[1] : live[2])) {
      tail->prefix[PASS - 1][tid] = sel_prefix[tid];
      tail->left[PASS - 1][tid] = sel_left[tid];
    }
    // ---- count the next bits of the keys in those buckets
    constexpr uint32_t kShift = PASS == 1 ? 20u : 10u;
    for_each_key(a, t0, t1, [&](uint32_t key) {
      const uint32_t high = key >> kShift, d = (key >> (kShift - 10u)) & (kSub - 1u);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (high == prefix[k]) atomicAdd(&hist[k * kSub + d], 1u);
        if (PASS == 2) below[k] += (uint32_t)(high < prefix[k]);
      }
    });
    __syncthreads();
    CNT* dst = (PASS == 1 ? mid_hist<CNT>(a, b) : low_hist<CNT>(a, b)) + tid;
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[k * kSub] = (CNT)hist[k * kSub + tid];
    if constexpr (PASS == 2) {
      uint32_t inc[3], all[3];
      block_scan<3>(below, inc, all, tot, lane, wave);
      if (tid < 3) tail->below[b][tid] = tid == 0 ? all[0] : tid == 1 ? all[1] : all[2];
    }
  }
}

// The cuts' keys, and for every workgroup what the tokens in front of its own add up to.  One workgroup.
template <typename CNT>
__global__ __launch_bounds__(kThreads) void long_settle_kernel(LongArgs a) {
  __shared__ uint32_t tot[3][kSelectWaves];
  __shared__ uint32_t sel_digit[3], sel_left[3], sel_same[3];
  __shared__ uint32_t less[3][kMaxParts];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const Tail* tail = tail_of<CNT>(a);
  const bool live[3] = {a.cut[0] < a.tokens, a.cut[1] < a.tokens, a.cut[2] < a.tokens};
  uint32_t own[3] = {0, 0, 0}, inc[3], all[3];
#pragma unroll 4
  for (uint32_t p = 0; p < a.parts; ++p) {
    const CNT* src = low_hist<CNT>(a, p) + tid;
#pragma unroll
    for (int k = 0; k < 3; ++k) own[k] += src[k * kSub];
  }
  block_scan<3>(own, inc, all, tot, lane, wave);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t want = tail->left[1][k];
    if (live[k] && inc[k] > want && inc[k] - own[k] <= want) {
      sel_digit[k] = tid;
      sel_left[k] = want - (inc[k] - own[k]);
      sel_same[k] = own[k];
    }
  }
  __syncthreads();
  // a wave per (workgroup, cut): its keys in front of the cut's key
  for (uint32_t i = wave; i < 3u * a.parts; i += kSelectWaves) {
    const uint32_t p = i / 3u, k = i - 3u * p;
    if (!(k == 0 ? live[0] : k == 1 ? live[1] : live[2])) continue;
    const uint32_t digit = sel_digit[k];
    const CNT* src = low_hist<CNT>(a, p) + k * kSub;
    uint32_t s = 0;
#pragma unroll
    for (uint32_t j = 0; j < kSub / kWaveSize; ++j) {
      const uint32_t d = j * kWaveSize + lane;
      const uint32_t h = src[d];
      s += d < digit ? h : 0u;
    }
    s = wave_inclusive_scan(s);
    if (lane == 63) less[k][p] = s + tail->below[p][k];
  }
  __syncthreads();
  uint32_t key = 0, quota = 0, before = 0, ahead = 0, tied = 0;
  if (wave < 3) {                                             // wave = cut, lane = workgroup
    const bool on = wave == 0 ? live[0] : wave == 1 ? live[1] : live[2];
    if (on) {
      key = (tail->prefix[1][wave] << 10) | sel_digit[wave];
      quota = sel_left[wave];
      tied = sel_same[wave] > 1u;
      const uint32_t same = lane < a.parts ? (uint32_t)low_hist<CNT>(a, lane)[wave * kSub + sel_digit[wave]] : 0u;
      before = wave_inclusive_scan(same) - same;
      const uint32_t admitted = quota > before ? min(quota - before, same) : 0u;
      const uint32_t in_front = (lane < a.parts ? less[wave][lane] : 0u) + admitted;
      ahead = wave_inclusive_scan(in_front) - in_front;
    } else {
      ahead = min(lane * a.per, a.tokens);                    // every token lies in front of this cut
    }
  }
  __syncthreads();                                            // everything has been read: the results may go over it
  if (tid == 0) tot[0][0] = 0u;
  __syncthreads();
  if (wave < 3 && lane == 0 && tied) atomicOr(&tot[0][0], 1u);
  __syncthreads();
  if (wave < 3 && lane < a.parts) {
    Part* p = reinterpret_cast<Part*>(a.result + part_offset(a.result, a.result_step, lane));
    p->key[wave] = key; p->quota[wave] = quota; p->same[wave] = before; p->ahead[wave] = ahead;
    if (wave == 0) p->tied = tot[0][0];
  }
}

// Widths, and with PLAN the card's tables, header and pads.  Every thread takes four consecutive tokens a turn.
template <bool PLAN>
__global__ __launch_bounds__(kThreads) void long_write_kernel(LongArgs a, uint8_t* __restrict__ bits, PlanArgs plan) {
  __shared__ uint32_t tot[2][3][kSelectWaves];
  __shared__ Part part;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, b = blockIdx.x;
  const uint32_t t0 = b * a.per, t1 = min(t0 + a.per, a.tokens);
  const bool live[3] = {a.cut[0] < a.tokens, a.cut[1] < a.tokens, a.cut[2] < a.tokens};
  if (tid < sizeof(Part) / 4u)
    reinterpret_cast<uint32_t*>(&part)[tid] =
        reinterpret_cast<const uint32_t*>(a.result + part_offset(a.result, a.result_step, b))[tid];
  __syncthreads();                                            // read by now: the stores below may go over it
  const bool tied = uniform(part.tied) != 0u;
  uint32_t key[3], quota[3], same[3], ahead[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    key[k] = uniform(part.key[k]); quota[k] = uniform(part.quota[k]);
    same[k] = uniform(part.same[k]); ahead[k] = uniform(part.ahead[k]);
  }
  uint32_t* slot_out = PLAN ? reinterpret_cast<uint32_t*>(plan.card + plan.g.off_slot) : nullptr;
  uint32_t* order_out = PLAN ? reinterpret_cast<uint32_t*>(plan.card + plan.g.off_order) : nullptr;
  const bool words_ok = bits == nullptr || (reinterpret_cast<uintptr_t>(bits) & 3u) == 0u;      // per is a multiple of 4

  for (uint32_t base = t0; base < t1; base += 4u * kThreads) {
    const uint32_t t = base + 4u * tid;
    const uint32_t n = t < t1 ? min(t1 - t, 4u) : 0u;
    uint32_t x[4];
    if (a.aligned && n == 4u) {
      const float4 s = *reinterpret_cast<const float4*>(a.scores + t);
      x[0] = rank_key(s.x); x[1] = rank_key(s.y); x[2] = rank_key(s.z); x[3] = rank_key(s.w);
    } else {
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i) x[i] = i < n ? rank_key(a.scores[t + i]) : 0u;
    }
    uint32_t run[3] = {0, 0, 0};
    if (tied) {                                               // tokens with a cut's key are admitted by increasing index
      uint32_t eq[3] = {0, 0, 0}, inc[3], all[3];
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) eq[k] += (uint32_t)(i < n && live[k] && x[i] == key[k]);
      block_scan<3>(eq, inc, all, tot[0], lane, wave);
#pragma unroll
      for (int k = 0; k < 3; ++k) { run[k] = same[k] + inc[k] - eq[k]; same[k] += all[k]; }
    }
    uint32_t cls[4], at_least[3] = {0, 0, 0};                 // own tokens in front of cuts 2, 1, 0: class >= 1, 2, 3
#pragma unroll
    for (uint32_t i = 0; i < 4u; ++i) {
      cls[i] = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const bool is_eq = x[i] == key[k];
        const bool in_front = !live[k] || x[i] < key[k] || (is_eq && (!tied ? quota[k] != 0u : run[k] < quota[k]));
        run[k] += is_eq;
        cls[i] += in_front;
      }
      at_least[0] += (uint32_t)(i < n && cls[i] >= 1u);
      at_least[1] += (uint32_t)(i < n && cls[i] >= 2u);
      at_least[2] += (uint32_t)(i < n && cls[i] >= 3u);
    }
    const uint32_t widths = (2u << cls[0]) | ((2u << cls[1]) << 8) | ((2u << cls[2]) << 16) | ((2u << cls[3]) << 24);
    if (bits != nullptr && n != 0u) {
      if (words_ok && n == 4u) *reinterpret_cast<uint32_t*>(bits + t) = widths;
      else for (uint32_t i = 0; i < n; ++i) bits[t + i] = (uint8_t)(widths >> (8u * i));
    }
    if constexpr (PLAN) {
      uint32_t inc[3], all[3];
      block_scan<3>(at_least, inc, all, tot[1], lane, wave);
      // tokens in front of this thread's that are of class >= 1, 2, 3, and from them the next free slot of every class
      const uint32_t f1 = ahead[2] + inc[0] - at_least[0], f2 = ahead[1] + inc[1] - at_least[1], f3 = ahead[0] + inc[2] - at_least[2];
      uint32_t next[4] = {t - f1, f1 - f2, f2 - f3, f3};
      uint32_t slot[4];
#pragma unroll
      for (uint32_t i = 0; i < 4u; ++i) {
        const uint32_t c = cls[i];
        slot[i] = c == 0u ? next[0] : c == 1u ? next[1] : c == 2u ? next[2] : next[3];
        next[0] += (c == 0u); next[1] += (c == 1u); next[2] += (c == 2u); next[3] += (c == 3u);
        if (i < n) order_out[(c == 0u ? 0u : c == 1u ? plan.g.base[1] : c == 2u ? plan.g.base[2] : plan.g.base[3]) + slot[i]] = t + i;
      }
      if (n == 4u) {
        *reinterpret_cast<u32x4*>(slot_out + t) = (u32x4){slot[0], slot[1], slot[2], slot[3]};
        *reinterpret_cast<uint32_t*>(plan.card + plan.g.off_bits + t) = widths;
      } else {
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) if (i < n) { slot_out[t + i] = slot[i]; plan.card[plan.g.off_bits + t + i] = (uint8_t)(widths >> (8u * i)); }
      }
      ahead[2] += all[0]; ahead[1] += all[1]; ahead[0] += all[2];
    }
    if (base + 4u * kThreads < t1) __syncthreads();           // the wave totals are written again
  }
  // by the last workgroup: its Part may reach into the pad behind the slot table when it has few tokens, and it has read it
  if (PLAN && b + 1u == a.parts) write_header_and_pads(plan.card, plan.header, plan.pads, 0u, tid);
}

template <typename CNT>
hipError_t launch_chain(const LongArgs& a, uint8_t* bits, const PlanArgs* plan, hipStream_t stream) {
  const dim3 grid(a.parts), block(kThreads);
  hipLaunchKernelGGL((long_pass_kernel<0, CNT>), grid, block, 0, stream, a);
  hipLaunchKernelGGL((long_pass_kernel<1, CNT>), grid, block, 0, stream, a);
  hipLaunchKernelGGL((long_pass_kernel<2, CNT>), grid, block, 0, stream, a);
  hipLaunchKernelGGL(long_settle_kernel<CNT>, dim3(1), block, 0, stream, a);
  if (plan) hipLaunchKernelGGL(long_write_kernel<true>, grid, block, 0, stream, a, bits, *plan);
  else hipLaunchKernelGGL(long_write_kernel<false>, grid, block, 0, stream, a, bits, PlanArgs());
  return hipGetLastError();
}

uint32_t round_up(uint64_t x, uint32_t m) { return (uint32_t)((x + m - 1) / m * m); }

}  // namespace

// tokens > 32768 (the scratch arithmetic needs it)
hipError_t launch_assign_long(const float* scores, uint32_t tokens, const uint32_t cuts[3], uint8_t* bits, hipStream_t stream) {
  LongArgs a;
  a.scores = scores;
  a.tokens = tokens;
  for (int k = 0; k < 3; ++k) a.cut[k] = cuts[k];
  a.aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0;
  // the bits array is all the scratch there is: as many workgroups as their histograms fit into it
  const uint64_t room = (uint64_t)tokens - 15u - sizeof(Tail);
  uint64_t parts = room / part_bytes<uint16_t>();
  if (parts > kMaxParts) parts = kMaxParts;
  a.per = round_up((tokens + parts - 1) / parts, 4u);
  const bool wide = a.per > 0xFFFFu;                          // a workgroup's counts beyond 16 bits: only with all 64 of them
  a.parts = (tokens + a.per - 1) / a.per;
  const uint64_t base = reinterpret_cast<uint64_t>(bits);
  a.hist = bits + (((base + 15u) & ~(uint64_t)15u) - base);
  a.result = bits;
  a.result_step = a.per;
  return wide ? launch_chain<uint32_t>(a, bits, nullptr, stream) : launch_chain<uint16_t>(a, bits, nullptr, stream);
}

hipError_t launch_assign_plan_long(const float* scores, const uint32_t cuts[3], uint8_t* bits, const CardGeom& geom,
                                   const qkv_card_header_t& header, uint8_t* card, hipStream_t stream) {
  PlanArgs plan;
  plan.g = geom;
  plan.header = header;
  plan.pads = make_pad_table(geom);
  plan.card = card;
  plan.share_waves = 0;
  LongArgs a;
  a.scores = scores;
  a.tokens = geom.tokens;
  for (int k = 0; k < 3; ++k) a.cut[k] = cuts[k];
  a.aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0;
  // slot and order tables, 8 bytes per token, are the scratch: 8192 tokens per workgroup, more beyond 512K tokens
  a.per = round_up(((uint64_t)geom.tokens + kMaxParts - 1) / kMaxParts, 64u);
  if (a.per < 8192u) a.per = 8192u;
  a.parts = (geom.tokens + a.per - 1) / a.per;
  a.hist = card + geom.off_slot;
  a.result = card + geom.off_slot;
  a.result_step = 4ull * a.per;
  return a.per > 0xFFFFu ? launch_chain<uint32_t>(a, bits, &plan, stream) : launch_chain<uint16_t>(a, bits, &plan, stream);
}

}  // namespace qkv
