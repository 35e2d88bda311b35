// assign.hip — bit-width assignment from per-token scores (paper Sec. 3.3: the combined
// score S(t) decides b(t) under a memory budget), the planning of a card from the same scores
// (Sec. 4.2.1: bit-width vector, slots, header), and the histogram of a bits vector.
//
// Ranking rule: tokens ordered by (score descending, index ascending), scores compared in
// the IEEE total order.  The first cut[0] tokens get 16 bits, up to cut[1] 8 bits, up to
// cut[2] 4 bits, the rest 2.  No sort is needed: for each cut a radix select over the 32-bit
// order keys finds the key of the token at that rank and how many tokens lie strictly
// before it; tokens whose key equals the cut key are then admitted by increasing index until
// the cut is full (a stable block-wide prefix count).  One workgroup of 1024 threads does the
// selection; thread i owns the consecutive tokens [i * per, (i + 1) * per).
//
// What this kernel costs is set by two things, neither of them memory: it runs once per launch,
// so every line of its code is fetched cold, and its sixteen waves share the issue slots of one
// compute unit.  Hence: a thread keeps its keys in registers, and the kernel is instantiated per
// number of keys per thread (1, 2, 4, ... 32, chosen from the token count), so that a launch
// touches only the code of its own size; the passes after the first are one rolled loop; later
// passes test a key against all three cut prefixes and skip the counting code for waves that hold no
// match; a wave without ties needs three comparisons per key for the widths.  Longer sequences
// (kRankedMax, kPlanMax): assign_long.hip.
//
// Planning variant (PLAN): once the cut keys are known every thread knows the widths of its own
// tokens, so a block-wide prefix count of the classes gives the stable slots, order[] and the
// bits copy, and the header follows - scores to a planned card in one launch instead of three
// (allocator, classification, and the gaps between them).  The launch has several workgroups:
// each repeats the whole selection by itself (no workgroup talks to another) and then writes the
// tables of its own share of at most 2048 consecutive tokens.  A share's entries of order[] are
// four contiguous runs, one per class; they, the slots and the widths are put together in LDS and
// leave as whole lines.
#include "qkv_common.h"
#include "qkv_plan.h"
#include "qkv_select.h"

namespace qkv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = kSelectThreads;
constexpr int kWaves = kSelectWaves;
constexpr uint32_t kTop = 4096, kSub = 1024; // buckets of the first pass, and of the two later ones for each cut
constexpr uint32_t kTopCopies = 4;           // of the first pass's histogram, against same-word atomics: real scores share sign and exponent
constexpr uint32_t kByteCopies = 16;         // the same for a first pass of 8 bits
// Longest sequences one workgroup's registers take; assign_long.hip goes on.  Widths alone, one workgroup against the chain
// of launches there: 12 / 24 us at 16384 tokens, 21 / 27 at 32768.  With planning the line lies at the last size of 16
// keys per thread: with 32 one workgroup is little faster without ties and much slower with (scores without ties: 16385 tokens
// 21.5 / 24.4 us, 20000 23.0 / 24.6, 24000 23.4 / 24.7, 28000 25.0 / 25.3, 32768 26.1 / 25.3; fifty different scores: 28.2 / 26.5,
// 30.8 / 26.4, 31.3 / 26.7, 34.5 / 26.9, 35.6 / 26.8).
constexpr uint32_t kRankedMax = 32768;
constexpr uint32_t kPlanMax = 16384;
constexpr uint32_t kShareTokens = 2048;      // tokens whose tables one workgroup writes

// Counts a key in the one of three histograms of `size` buckets, a power of two, whose cut its higher bits (from `above` on) lead to; the
// three only's differ, or are all ones, which no key's higher bits are.  Many waves hold no key of any cut, so which one it is gets worked out behind the
// branch, and the compiler is kept from doing it in front (8192 tokens without ties 7.56 us so and 7.25, 12000 spread over all exponents 10.7
// and 9.7; with three branches, one a cut, 8.0 and 10.2).
__device__ __forceinline__ void count_key(uint32_t* hist, uint32_t size, uint32_t key, uint32_t shift, uint32_t above, uint32_t only0,
                                          uint32_t only1, uint32_t only2, bool own) {
  uint32_t high = key >> above;
  const bool any = own && (high == only0 || high == only1 || high == only2);
  if (__builtin_amdgcn_ballot_w64(any) != 0ull) {
    asm volatile("" : "+v"(high));
    if (any) atomicAdd(&hist[((key >> shift) & (size - 1u)) + (high == only1 ? size : high == only2 ? 2u * size : 0u)], 1u);
  }
}

// T <= KPT * 1024: thread tid owns the tokens [tid * KPT, tid * KPT + KPT) and keeps their keys in registers.
// PLAN: also write slot[], order[], the bits copy, header and pads of plan->card; `bits` may then be null.
template <int KPT, bool PLAN>
__device__ __forceinline__ void ranked_body(const float* __restrict__ scores, uint32_t T, uint32_t cut0, uint32_t cut1,
                                            uint32_t cut2, uint8_t* __restrict__ bits, bool aligned, const PlanArgs* plan) {
  // Up to 8 keys per thread four passes of 8 bits, more keys 12, 10 and 10 bits: a pass less to make over the keys, but
  // more buckets to clear and add up, and fewer copies of them, which scores that crowd together feel (see lanes_crowd).
  // Widths alone, us, four passes and three, for uniform scores / a constant / half of them zero: 4096 tokens 6.4 / 16.5 / 6.3
  // and 6.8 / 14.3 / 7.0, 8192 8.4 / 28.7 / 8.3 and 8.3 / 23.2 / 9.5, 16384 13.6 / 54.0 / 13.3 and 12.4 / 42.2 / 14.2, 32768
  // 26.3 / 108 / 25.8 and 22.3 / 82.2 / 25.8.
  constexpr bool kBytes = KPT <= 8;
  // first pass: bucket d, copy c at word [d * copies + c]; later the other passes' histograms; then the stage
  __shared__ u32x4 wide4[(kBytes ? 256u * kByteCopies + 6u * 256u : kTop * kTopCopies) / 4u];
  __shared__ uint32_t sel_prefix[3];                    // key bits fixed so far
  __shared__ uint32_t sel_left[3];                      // rank still to descend inside the current bucket
  __shared__ uint32_t sel_same[3];                      // keys equal to the cut key
  __shared__ __attribute__((aligned(16))) uint32_t wave_tot[3][kWaves];
  __shared__ __attribute__((aligned(16))) uint32_t wave_cls[3][kWaves];
  uint32_t* wide = reinterpret_cast<uint32_t*>(wide4);
  uint32_t* hist2 = wide + 256u * kByteCopies;          // 8-bit passes: two sets of [cut][256], one cleared while the other is searched
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  const uint32_t cut[3] = {cut0, cut1, cut2};
  // A cut equal to T has no token at that rank: every token lies before it, handled without a key.
  // Cuts do not decrease, so live[2] implies live[1] implies live[0].
  const bool live[3] = {cut0 < T, cut1 < T, cut2 < T};

  const uint32_t t0 = min(tid * (uint32_t)KPT, T);
  const uint32_t n_own = min(t0 + (uint32_t)KPT, T) - t0;
  uint32_t keys[KPT];
  if (KPT % 4 == 0 && aligned && n_own == (uint32_t)KPT) {          // 128-bit loads
#pragma unroll
    for (int i = 0; i < KPT; i += 4) {
      const float4 f = *reinterpret_cast<const float4*>(scores + t0 + i);
      keys[i] = rank_key(f.x); keys[i + 1] = rank_key(f.y); keys[i + 2] = rank_key(f.z); keys[i + 3] = rank_key(f.w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < KPT; ++i) keys[i] = ((uint32_t)i < n_own) ? rank_key(scores[t0 + i]) : 0u;
  }

  if constexpr (kBytes) {
    // ---- pass 0: one histogram of the top byte, shared by the three cuts
    wide4[tid] = (u32x4)(0u);                             // 256 * 16 words = 1024 x 16 bytes
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      if ((uint32_t)i < n_own) atomicAdd(&wide[(keys[i] >> 24) * kByteCopies + (lane & (kByteCopies - 1u))], 1u);
    __syncthreads();
    if (tid < 256) {
      uint32_t s = 0;
#pragma unroll
      for (int i = 0; i < kByteCopies; ++i) s += wide[tid * kByteCopies + ((i + tid) & (kByteCopies - 1u))];
      hist2[tid] = s;
    } else if (tid < 4 * 256) {
      hist2[768u + tid - 256u] = 0;          // the set the next pass counts into
    }
    __syncthreads();
    if (wave < 3 && live[wave]) {
      uint32_t left = cut[wave], same;
      const uint32_t d = find_bucket(hist2, lane, left, same);
      if (lane == 0) { sel_prefix[wave] = d << 24; sel_left[wave] = left; }
    }
    __syncthreads();

    // ---- passes 1..3: per cut, only the keys inside its bucket so far.  Cuts whose prefixes are still the
    // same count the same keys: they share the histogram of the first of them (rep).
#pragma unroll 1
    for (int pass = 1; pass < 4; ++pass) {
      const uint32_t shift = 24u - 8u * (uint32_t)pass;
      const uint32_t pre0 = uniform(sel_prefix[0]), pre1 = uniform(sel_prefix[1]), pre2 = uniform(sel_prefix[2]);
      const uint32_t rep1 = (live[0] && pre1 == pre0) ? 0u : 1u;
      const uint32_t rep2 = (live[0] && pre2 == pre0) ? 0u : (live[1] && pre2 == pre1) ? 1u : 2u;
      // what a key's higher bits are compared with; no key's are all ones after the shift.  The three differ, so a key is counted once.
      const uint32_t only0 = live[0] ? pre0 >> (shift + 8u) : 0xFFFFFFFFu;
      const uint32_t only1 = live[1] && rep1 == 1u ? pre1 >> (shift + 8u) : 0xFFFFFFFFu;
      const uint32_t only2 = live[2] && rep2 == 2u ? pre2 >> (shift + 8u) : 0xFFFFFFFFu;
      uint32_t* hist = hist2 + 768u * (pass & 1);         // cleared during the previous search
#pragma unroll
      for (int i = 0; i < KPT; ++i) count_key(hist, 256u, keys[i], shift, shift + 8u, only0, only1, only2, (uint32_t)i < n_own);
      __syncthreads();
      if (wave < 3) {
        if (live[wave]) {
          const uint32_t from = wave == 0 ? 0u : wave == 1 ? rep1 : rep2;
          uint32_t left = sel_left[wave], same;
          const uint32_t d = find_bucket(hist + 256u * from, lane, left, same);
          if (lane == 0) { sel_prefix[wave] |= d << shift; sel_left[wave] = left; sel_same[wave] = same; }
        }
      } else if (wave < 15) {                             // meanwhile the other set is cleared for the next pass
        const uint32_t i = tid - 3u * kWaveSize;          // 0 .. 767
        hist2[768u * ((pass & 1) ^ 1) + i] = 0;
      }
      __syncthreads();
    }
  } else {
    // ---- pass 0: one histogram of the top 12 bits, shared by the three cuts; thread tid sums buckets 4 tid .. + 3
#pragma unroll
    for (uint32_t i = 0; i < kTop * kTopCopies / 4u / kThreads; ++i) wide4[i * kThreads + tid] = (u32x4)(0u);
    __syncthreads();
    if (lanes_crowd(keys[0] >> 20, n_own != 0u)) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) add_crowded(wide, (keys[i] >> 20) * kTopCopies, (uint32_t)i < n_own, lane);
    } else {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if ((uint32_t)i < n_own) atomicAdd(&wide[(keys[i] >> 20) * kTopCopies + (lane & (kTopCopies - 1u))], 1u);
    }
    __syncthreads();
    {
      uint32_t c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { const u32x4 h = wide4[4u * tid + i]; c[i] = h.x + h.y + h.z + h.w; }
      const uint32_t own[1] = {c[0] + c[1] + c[2] + c[3]};
      uint32_t inc[1], all[1];
      block_scan<1>(own, inc, all, wave_tot, lane, wave);         // every bucket has been read behind its barrier
#pragma unroll
      for (uint32_t i = 0; i < 2u * 3u; ++i) wide[i * kSub + tid] = 0u;      // the histograms of both later passes
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        uint32_t left = cut[k] - (inc[0] - own[0]);
        if (live[k] && inc[0] > cut[k] && inc[0] - own[0] <= cut[k]) {        // exactly one thread
          uint32_t d = 0;
          if (left >= c[0]) { left -= c[0]; d = 1; if (left >= c[1]) { left -= c[1]; d = 2; if (left >= c[2]) { left -= c[2]; d = 3; } } }
          sel_prefix[k] = 4u * tid + d;
          sel_left[k] = left;
        }
      }
    }
    __syncthreads();

    // ---- passes 1 and 2, 10 bits each: per cut, only the keys inside its bucket so far.  Cuts whose prefixes are still the
    // same share the histogram of the first of them (rep).
#pragma unroll 1
    for (uint32_t pass = 0; pass < 2u; ++pass) {
      uint32_t pre[3], want[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        pre[k] = live[k] ? uniform(sel_prefix[k]) : 0xFFFFFFFFu;              // no key has that prefix
        want[k] = uniform(sel_left[k]);
      }
      const uint32_t shift = pass == 0u ? 20u : 10u;
      const uint32_t rep1 = pre[1] == pre[0] ? 0u : 1u, rep2 = pre[2] == pre[0] ? 0u : pre[2] == pre[1] ? 1u : 2u;
      uint32_t* hist = wide + pass * 3u * kSub;
      const uint32_t only1 = rep1 == 1u ? pre[1] : 0xFFFFFFFFu, only2 = rep2 == 2u ? pre[2] : 0xFFFFFFFFu;
#pragma unroll
      for (int i = 0; i < KPT; ++i) count_key(hist, kSub, keys[i], shift - 10u, shift, pre[0], only1, only2, (uint32_t)i < n_own);
      __syncthreads();
      const uint32_t own[3] = {hist[tid], hist[rep1 * kSub + tid], hist[rep2 * kSub + tid]};
      uint32_t inc[3], all[3];
      block_scan<3>(own, inc, all, wave_tot, lane, wave);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (live[k] && inc[k] > want[k] && inc[k] - own[k] <= want[k]) {
          sel_prefix[k] = (pre[k] << 10) | tid;
          sel_left[k] = want[k] - (inc[k] - own[k]);
          sel_same[k] = own[k];
        }
      }
      __syncthreads();
    }
  }

  // Now sel_prefix[c] is the key at rank cut[c], sel_same[c] the number of tokens with exactly that key and
  // sel_left[c] how many of those still belong before the cut.
  uint32_t keyc[3], quota[3];
  bool unique = true;               // every cut key occurs once: then it is the cut token's own, and no tie rule is needed
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    keyc[c] = uniform(sel_prefix[c]); quota[c] = uniform(sel_left[c]);
    unique = unique && (!live[c] || uniform(sel_same[c]) == 1u);
  }
  uint32_t run[3] = {0, 0, 0};
  bool no_ties = true;
  if (!unique) {
    uint32_t eq[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
#pragma unroll
      for (int c = 0; c < 3; ++c) eq[c] += ((uint32_t)i < n_own && live[c] && keys[i] == keyc[c]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t inc = wave_inclusive_scan(eq[c]);
      run[c] = inc - eq[c];
      if (lane == 63) wave_tot[c][wave] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) run[c] += waves_below(scan_wave_totals(wave_tot[c], lane), wave);
    // A wave none of whose keys equals a cut key needs no tie rule either.
    no_ties = __builtin_amdgcn_ballot_w64((eq[0] | eq[1] | eq[2]) != 0u) == 0ull;
  }
  // Class of a key: how many of the three cuts it lies before (0..3 for 2, 4, 8, 16 bits).  The cut keys do not
  // decrease and a token admitted at one cut is admitted at the later ones, so the three answers just add up.
  auto class_of_key = [&](uint32_t key) -> uint32_t {
    uint32_t c = 0;
    if (no_ties) {                  // three comparisons per key
#pragma unroll
      for (int k = 0; k < 3; ++k) c += (!live[k] || key < keyc[k]);
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (!live[k]) { ++c; continue; }
        const bool is_eq = key == keyc[k];
        c += (key < keyc[k] || (is_eq && run[k] < quota[k]));
        run[k] += is_eq;
      }
    }
    return c;
  };
  auto width_of = [&](uint32_t key) -> uint32_t { return 2u << class_of_key(key); };

  if constexpr (!PLAN) {
    if (KPT % 8 == 0 && aligned && n_own == (uint32_t)KPT) {       // 8 widths per 64-bit store
#pragma unroll
      for (int i = 0; i < KPT; i += 8) {
        uint64_t w = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) w |= (uint64_t)width_of(keys[i + j]) << (8 * j);
        *reinterpret_cast<uint64_t*>(bits + t0 + i) = w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if ((uint32_t)i < n_own) bits[t0 + i] = (uint8_t)width_of(keys[i]);
    }
  } else {
    // ---- the card's front matter.  Thread tid owns the consecutive tokens [t0, t0 + n_own), so exactly t0
    // tokens lie before them, and the classes among those follow from a block-wide prefix count.
    const CardGeom& g = plan->g;
    uint8_t* card = plan->card;
    uint8_t* bits_card = card + g.off_bits;
    uint32_t* slot_out = reinterpret_cast<uint32_t*>(card + g.off_slot);
    uint32_t* order_out = reinterpret_cast<uint32_t*>(card + g.off_order);
    const uint32_t w0 = blockIdx.x * plan->share_waves, w1 = min(w0 + plan->share_waves, (uint32_t)kWaves);
    const bool mine = wave >= w0 && wave < w1;            // whole waves
    uint32_t cls[(KPT + 15) / 16] = {};                   // the classes of the own tokens, 2 bits each
    uint32_t at_least[3] = {0, 0, 0};                     // own tokens of class >= 1, 2, 3
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      if ((uint32_t)i < n_own) {
        const uint32_t c = class_of_key(keys[i]);
        cls[i / 16] |= c << (2 * (i % 16));
        at_least[0] += (c >= 1u); at_least[1] += (c >= 2u); at_least[2] += (c >= 3u);
      }
    }
    const uint32_t own[3] = {at_least[0] - at_least[1], at_least[1] - at_least[2], at_least[2]};   // of 4, 8, 16 bits
    uint32_t before[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t inc = wave_inclusive_scan(own[c]);
      before[c] = inc - own[c];
      if (lane == 63) wave_cls[c][wave] = inc;
    }
    __syncthreads();
    // class runs of this workgroup's share inside order[]: first slot and length (classes 1..3 counted, class 0 the rest)
    uint32_t first[4], len[4];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t running = scan_wave_totals(wave_cls[c], lane);
      before[c] += waves_below(running, wave);
      first[c + 1] = waves_below(running, w0);
      len[c + 1] = waves_below(running, w1) - first[c + 1];
    }
    const uint32_t share_t0 = min(w0 * (uint32_t)(kWaveSize * KPT), T), share_t1 = min(w1 * (uint32_t)(kWaveSize * KPT), T);
    const uint32_t share_n = share_t1 - share_t0;         // <= kShareTokens
    first[0] = share_t0 - first[1] - first[2] - first[3];
    len[0] = share_n - len[1] - len[2] - len[3];
    const uint32_t at[4] = {0u, len[0], len[0] + len[1], len[0] + len[1] + len[2]};      // run starts inside the stage
    uint32_t* stage_order = wide;                         // kShareTokens entries each
    uint32_t* stage_slot = wide + kShareTokens;
    uint8_t* stage_bits = reinterpret_cast<uint8_t*>(wide + 2u * kShareTokens);
    if (mine) {
      // next free slot of every class for this thread's tokens; class 0 is what remains of the t0 tokens before
      uint32_t next[4] = {t0 - before[0] - before[1] - before[2], before[0], before[1], before[2]};
      const uint32_t lt0 = t0 - share_t0;
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        if ((uint32_t)i < n_own) {
          const uint32_t c = (cls[i / 16] >> (2 * (i % 16))) & 3u;
          const uint32_t s = (c == 0) ? next[0] : (c == 1) ? next[1] : (c == 2) ? next[2] : next[3];
          next[0] += (c == 0); next[1] += (c == 1); next[2] += (c == 2); next[3] += (c == 3);
          const uint32_t li = s + ((c == 0) ? at[0] - first[0] : (c == 1) ? at[1] - first[1] : (c == 2) ? at[2] - first[2]
                                                                                                     : at[3] - first[3]);
          stage_order[li] = t0 + i;
          stage_slot[lt0 + i] = s;
          stage_bits[lt0 + i] = (uint8_t)width_of_class((int)c);
        }
      }
    }
    __syncthreads();
    for (uint32_t i = tid; i < share_n; i += kThreads) slot_out[share_t0 + i] = stage_slot[i];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      for (uint32_t i = tid; i < len[c]; i += kThreads) order_out[g.base[c] + first[c] + i] = stage_order[at[c] + i];
    // widths: share_t0 is a multiple of 64, so the card's copy goes out in words; the caller's pointer may be odd
    const uint32_t* stage_words = reinterpret_cast<const uint32_t*>(stage_bits);
    const bool words_ok = bits == nullptr || (reinterpret_cast<uintptr_t>(bits) & 3u) == 0u;
    for (uint32_t i = tid; i < share_n / 4u; i += kThreads) {
      reinterpret_cast<uint32_t*>(bits_card + share_t0)[i] = stage_words[i];
      if (bits && words_ok) reinterpret_cast<uint32_t*>(bits + share_t0)[i] = stage_words[i];
    }
    for (uint32_t i = (share_n & ~3u) + tid; i < share_n; i += kThreads) {
      bits_card[share_t0 + i] = stage_bits[i];
      if (bits && words_ok) bits[share_t0 + i] = stage_bits[i];
    }
    if (bits && !words_ok)
      for (uint32_t i = tid; i < share_n; i += kThreads) bits[share_t0 + i] = stage_bits[i];
    // widths come from the allocator and the counts from the same cuts: nothing for the status word to report
    if (blockIdx.x == 0) write_header_and_pads(card, plan->header, plan->pads, 0u, tid);
  }
}

template <int KPT>
__global__ __launch_bounds__(kThreads) void ranked_assign_kernel(const float* __restrict__ scores, uint32_t T, uint32_t cut0,
                                                                 uint32_t cut1, uint32_t cut2, uint8_t* __restrict__ bits,
                                                                 bool aligned) {
  ranked_body<KPT, false>(scores, T, cut0, cut1, cut2, bits, aligned, nullptr);
}

template <int KPT>
__global__ __launch_bounds__(kThreads) void assign_plan_kernel(const float* __restrict__ scores, uint32_t cut0, uint32_t cut1,
                                                               uint32_t cut2, uint8_t* __restrict__ bits, bool aligned,
                                                               PlanArgs plan) {
  ranked_body<KPT, true>(scores, plan.g.tokens, cut0, cut1, cut2, bits, aligned, &plan);
}

__global__ __launch_bounds__(256) void count_kernel(const uint8_t* __restrict__ bits, uint64_t T,
                                                    unsigned long long* __restrict__ counts4) {
  __shared__ uint32_t part[4];
  if (threadIdx.x < 4) part[threadIdx.x] = 0;
  __syncthreads();
  uint32_t cnt[4] = {0, 0, 0, 0};
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < T; t += stride) {
    const uint32_t b = bits[t];
    cnt[0] += (b == 2); cnt[1] += (b == 4); cnt[2] += (b == 8); cnt[3] += (b == 16);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) if (cnt[c]) atomicAdd(&part[c], cnt[c]);
  __syncthreads();
  if (threadIdx.x < 4 && part[threadIdx.x]) atomicAdd(&counts4[threadIdx.x], (unsigned long long)part[threadIdx.x]);
}

__global__ void zero4_kernel(unsigned long long* p) {
  if (threadIdx.x < 4) p[threadIdx.x] = 0;
}

}  // namespace

namespace {
// Keys per thread of the ranked kernels: the smallest of 1, 2, 4, 8, 16, 32 that covers `tokens` with 1024 threads.
uint32_t keys_per_thread(uint32_t tokens) {
  uint32_t kpt = 1;
  while (kpt * kThreads < tokens) kpt *= 2;
  return kpt;
}
}  // namespace

hipError_t launch_assign(const float* scores, uint32_t tokens, const uint32_t cuts[3], uint8_t* bits,
                         hipStream_t stream) {
  const dim3 grid(1), block(kThreads);
  const bool aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0 && reinterpret_cast<uintptr_t>(bits) % 8 == 0;
#define QKV_LAUNCH_ASSIGN(K) \
  hipLaunchKernelGGL(ranked_assign_kernel<K>, grid, block, 0, stream, scores, tokens, cuts[0], cuts[1], cuts[2], bits, aligned)
  if (tokens > kRankedMax) {
    return launch_assign_long(scores, tokens, cuts, bits, stream);
  } else {
    switch (keys_per_thread(tokens)) {
      case 1: QKV_LAUNCH_ASSIGN(1); break;
      case 2: QKV_LAUNCH_ASSIGN(2); break;
      case 4: QKV_LAUNCH_ASSIGN(4); break;
      case 8: QKV_LAUNCH_ASSIGN(8); break;
      case 16: QKV_LAUNCH_ASSIGN(16); break;
      default: QKV_LAUNCH_ASSIGN(32); break;
    }
  }
#undef QKV_LAUNCH_ASSIGN
  return hipGetLastError();
}

hipError_t launch_assign_plan(const float* scores, const uint32_t cuts[3], uint8_t* bits, const CardGeom& geom,
                              const qkv_card_header_t& header, uint8_t* card, hipStream_t stream) {
  const uint32_t tokens = geom.tokens;
  if (tokens > kPlanMax) return launch_assign_plan_long(scores, cuts, bits, geom, header, card, stream);
  PlanArgs plan;
  plan.g = geom;
  plan.header = header;
  plan.pads = make_pad_table(geom);
  plan.card = card;
  const bool aligned = reinterpret_cast<uintptr_t>(scores) % 16 == 0;
  // a share is whole waves and at most kShareTokens tokens
  const uint32_t kpt = keys_per_thread(tokens);
  uint32_t share_waves = kShareTokens / (kpt * kWaveSize);             // >= 2 since kpt <= 16
  if (share_waves > (uint32_t)kWaves) share_waves = kWaves;
  const uint32_t used_waves = ((tokens + kpt - 1) / kpt + kWaveSize - 1) / kWaveSize;
  plan.share_waves = share_waves;
  const dim3 grid((used_waves + share_waves - 1) / share_waves), block(kThreads);
#define QKV_LAUNCH_PLAN(K) \
  hipLaunchKernelGGL(assign_plan_kernel<K>, grid, block, 0, stream, scores, cuts[0], cuts[1], cuts[2], bits, aligned, plan)
  switch (kpt) {
    case 1: QKV_LAUNCH_PLAN(1); break;
    case 2: QKV_LAUNCH_PLAN(2); break;
    case 4: QKV_LAUNCH_PLAN(4); break;
    case 8: QKV_LAUNCH_PLAN(8); break;
    default: QKV_LAUNCH_PLAN(16); break;
  }
#undef QKV_LAUNCH_PLAN
  return hipGetLastError();
}

hipError_t launch_count(const uint8_t* bits, uint64_t tokens, unsigned long long* counts4, hipStream_t stream) {
  hipLaunchKernelGGL(zero4_kernel, dim3(1), dim3(64), 0, stream, counts4);
  uint64_t blocks = (tokens + 256 * 16 - 1) / (256 * 16);
  if (blocks < 1) blocks = 1;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(count_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, bits, tokens, counts4);
  return hipGetLastError();
}

}  // namespace qkv
