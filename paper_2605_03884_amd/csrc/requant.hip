// requant.hip — one hop of a multi-hop chain without the dense cache in between (paper Sec. 3.2,
// challenge 3: a cache is forwarded from agent to agent; Sec. 4.2: a card is what travels).
//
// An agent that forwards a card at new bit widths would otherwise rebuild the dense fp16 cache
// (injection) and build the next card from it (card creation): 2 x (dense + card) bytes of traffic.
// Here every span of 32 values is read from the incoming card, decoded to what injection would write - 2-bit codes
// with its decoder, 4- and 8-bit codes with the attention kernel's, whose roundings are the same -, quantized with the
// card-creation kernel's quantizer and stored into the outgoing card; the
// dense values only ever exist in registers.  The result is, byte for byte, the card that creation
// would build from the injected cache.
//
// Work decomposition, two of them (the line between them stands in launch_requant).
//
// Windows of a width: a workgroup takes a window of up to 256 consecutive rows of one outgoing segment: of one
// plane, done for one or two planes, or, in short cards, of the segment as it lies, across planes.
// It looks the window's tokens up once (token through the outgoing card's
// order[], written by the classification kernel just before, old width and slot through the incoming
// card's tables), sorts them by old width into a list in LDS and cuts the list into rounds of at most 64
// spans of one old width; the four waves deal the rounds of all planes among themselves, each with the
// next round's loads in flight, and no round mixes widths.  The incoming card is read with plain loads
// whatever its size: rows that leave for different widths share lines, and windows that run at the
// same time find them in cache (nontemporal loads cost 26 % at 32K tokens).
//
// Windows of tokens (long cards): a workgroup takes 512 rows (plane, token) and sorts them by pair of old and new width.  Tokens
// in a row lie in a row in every segment of either card, so a window reads and writes every line once; its rounds are dealt out in the order
// of their middle rows, so that what shares a line is done at about the same time (16384 tokens of 512 planes, 6 to 4: rows past the L2 read
// 1.33 GB with windows of a width and 0.97, written 0.85 and 0.71, whole call 419 us and 375; in the order of the pairs it is a tenth slower than
// with windows of a width).  Vector issue is then 82 % of the kernel's time at 8K tokens, 3 to 2.5; at 32K, 6 to 4, it is 81 %, and reading and
// writing at once takes as long as the kernel (reading alone 393 us, writing alone 261, both 740).
//
// Spans that were 2-bit (most of a card at low budgets) are not expanded to 32 values at all: a group
// has four decoded values, in order, so its extrema follow from which codes occur, the quantizer runs
// on the four values, and the new codes are the old ones relabelled.
//
// Whole call with the new widths' assignment, 8K tokens, budget 3 to 2.5: 199 us with 64 rows of one plane sorted per wave and every span
// expanded to 32 values, 160 with windows of a width, 144 .. 146 with windows of tokens; 32K tokens, 6 to 4: 1162, 840 and 753 .. 764 us.
// Windows of a width: of 512 rows 171 and 936 us; without the next round's loads in flight 172 and 877; of 256 tokens over all
// widths at once, in the order of the pairs, 221 and 1137.
//
// The incoming card is untrusted: header and offsets are rebuilt and checked on the device, table
// entries are bounded before they are used.
#include "qkv_common.h"
#include "qkv_encode.h"
#include "qkv_plan.h"

namespace qkv {
namespace {

constexpr uint32_t kWindow = 256;             // rows of an outgoing segment that a workgroup looks up and sorts
constexpr uint32_t kMaxPlanes = 2;            // planes it does them for, at most
constexpr uint32_t kOld = 5;                  // old classes 0 .. 3, and 4: not placed by the incoming tables
constexpr uint32_t kMaxRounds = kWindow * 8u / kWaveSize + kOld;
constexpr uint32_t kMaxGridX = 65536;         // workgroups side by side: a grid's width in threads stays below 2^32 (2^21 layers times heads: 65536 and more)

struct RequantArgs {
  const uint8_t* card_in;
  uint64_t card_in_bytes;
  uint32_t layers, kv_heads, head_dim, group_size;
  uint64_t tokens;
  CardGeom out;                 // the outgoing card's geometry (host-known counts)
  uint8_t* card_out;
  uint32_t* status;             // may be null; holds the verdict on the incoming header already (classify_kernel)
  uint32_t windows[4];          // of every outgoing class: of one plane, or of all planes where the windows run across them
  uint32_t blocks;              // workgroups asked for (the grid may hold a few more)
  uint32_t window;              // rows of a window
  uint32_t group_planes;        // planes a workgroup does with one window; 0: the windows run across planes
  uint32_t stride;              // workgroups from those planes' first window to the next planes'
};

// Bits chosen from a where mask is 1, from b where it is 0: one instruction.
__device__ inline uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// Whether relabel_span2 applies to every lane's pair: a scale that is no negative number, and finite values (no other zero has a
// finite fourth value).
__device__ inline bool can_relabel(uint32_t old_pair) {
  const float s = half_bits_to_float(old_pair & 0xFFFFu), z = half_bits_to_float(old_pair >> 16);
  const uint32_t x3 = decode_pair(2.0f, 3.0f, s, z) >> 16;
  const bool odd = (old_pair & 0xFFFFu) > 0x7BFFu || (x3 & 0x7C00u) == 0x7C00u;
  return __builtin_amdgcn_ballot_w64(odd) == 0ull;
}

// 2-bit codes to W-bit codes.  The decoded values x_k = fp16(fma(k, scale, zero)) do not decrease with k (and are never
// -0: scale and zero are multiples of the smallest fp16 step), so the span's extrema are those of the smallest and the
// largest code that occurs; then four values go through the quantizer instead of 32.
template <int W, int GS>
__device__ __forceinline__ uint32_t relabel_span2(const uint32_t (&cw)[2], uint32_t old_pair, uint32_t (&out)[W]) {
  const float s = half_bits_to_float(old_pair & 0xFFFFu), z = half_bits_to_float(old_pair >> 16);
  const uint32_t x01 = decode_pair(0.0f, 1.0f, s, z), x23 = decode_pair(2.0f, 3.0f, s, z);
  constexpr uint32_t kLow = 0x55555555u;
  const uint32_t lo0 = cw[0] & kLow, lo1 = cw[1] & kLow, hi0 = (cw[0] >> 1) & kLow, hi1 = (cw[1] >> 1) & kLow;
  const bool any_hi = (hi0 | hi1) != 0u, all_hi = (hi0 & hi1) == kLow;
  // largest code: in the upper half if any high bit is set; there, or below, 1 more if such a code has its low bit set
  const uint32_t top_lo = any_hi ? ((lo0 & hi0) | (lo1 & hi1)) : (lo0 | lo1);
  const uint32_t x_top = any_hi ? x23 : x01;
  const uint32_t mx = top_lo != 0u ? x_top >> 16 : x_top & 0xFFFFu;
  // smallest code, the same way with "not set"
  const uint32_t bot_lo = all_hi ? (lo0 & lo1) : ((lo0 | hi0) & (lo1 | hi1));      // 1 wherever a code of the lower half has its low bit set, or is of the upper half
  const uint32_t x_bot = all_hi ? x23 : x01;
  const uint32_t mn = bot_lo == kLow ? x_bot >> 16 : x_bot & 0xFFFFu;
  uint32_t m = mn | (mn << 16), M = mx | (mx << 16);
  reduce_group<GS>(m, M);
  const uint32_t mn_h = m & 0xFFFFu;
  float neg_mn, inv;
  bool clamp;
  const uint32_t s_h = group_scale<W>(mn_h, M & 0xFFFFu, neg_mn, inv, clamp);
  // the four new codes, one per byte (those of values that do not occur may be anything)
  uint32_t u[4];
  u[0] = __float_as_uint(__builtin_fmaf(lo_plus(x01, neg_mn), inv, kMagic));
  u[1] = __float_as_uint(__builtin_fmaf(hi_plus(x01, neg_mn), inv, kMagic));
  u[2] = __float_as_uint(__builtin_fmaf(lo_plus(x23, neg_mn), inv, kMagic));
  u[3] = __float_as_uint(__builtin_fmaf(hi_plus(x23, neg_mn), inv, kMagic));
  if (clamp) {
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = min(u[k], kMagicBits + ((1u << W) - 1u));
  }
  const uint32_t c4 = __builtin_amdgcn_perm(__builtin_amdgcn_perm(u[3], u[2], 0x0C0C0400u),
                                            __builtin_amdgcn_perm(u[1], u[0], 0x0C0C0400u), 0x05040100u);
  if constexpr (W == 2) {
    const uint32_t rep = __builtin_amdgcn_perm(0u, 0xFFAA5500u, c4 & 0x03030303u);     // byte k: code k four times
    const uint32_t r0 = __builtin_amdgcn_perm(rep, rep, 0x00000000u), r1 = __builtin_amdgcn_perm(rep, rep, 0x01010101u);
    const uint32_t r2 = __builtin_amdgcn_perm(rep, rep, 0x02020202u), r3 = __builtin_amdgcn_perm(rep, rep, 0x03030303u);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t lo = i ? lo1 : lo0, hi = i ? hi1 : hi0;
      const uint32_t lo2 = lo | (lo << 1), hi2 = hi | (hi << 1);
      out[i] = bit_select(hi2, bit_select(lo2, r3, r2), bit_select(lo2, r1, r0));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint32_t a[4];                                // a[k]: the new codes of positions k, 4 + k, 8 + k, 12 + k
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = __builtin_amdgcn_perm(0u, c4, (cw[i] >> (2 * k)) & 0x03030303u);
      if constexpr (W == 4) {
        const uint32_t even = a[0] | (a[1] << 4), odd = a[2] | (a[3] << 4);
        out[2 * i] = __builtin_amdgcn_perm(odd, even, 0x05010400u);
        out[2 * i + 1] = __builtin_amdgcn_perm(odd, even, 0x07030602u);
      } else {
        const uint32_t p01 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), q01 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
        const uint32_t p23 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u), q23 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
        out[4 * i] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
        out[4 * i + 1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
        out[4 * i + 2] = __builtin_amdgcn_perm(q23, q01, 0x05040100u);
        out[4 * i + 3] = __builtin_amdgcn_perm(q23, q01, 0x07060302u);
      }
    }
  }
  return s_h | (mn_h << 16);
}

// A span as it lies in the incoming card: its codes (or its 32 raw values) and its pair.
struct OldSpan {
  uint32_t cw[16];
  uint32_t pair;
};

// Span `gsp` (row * spans per row + span) of old class CO.  By value: stores into one object out of several branches
// end up as one store to a computed place in scratch memory.
template <int CO, int G>
__device__ __forceinline__ OldSpan fetch_old(const uint8_t* card, const CardGeom& in, uint64_t gsp) {
  constexpr int GS = G / 32;
  constexpr int NW = CO == 3 ? 16 : (2 << CO);
  const uint8_t* src = card + (CO == 3 ? in.off_fp16 : in.off_codes[CO < 3 ? CO : 0]) + gsp * (4u * NW);
  OldSpan d;
  if constexpr (NW == 2) {
    const u32x2 v = card_load<true>(reinterpret_cast<const u32x2*>(src));
    d.cw[0] = v.x; d.cw[1] = v.y;
  } else {
#pragma unroll
    for (int h = 0; h < NW / 4; ++h) {
      const u32x4 v = card_load<true>(reinterpret_cast<const u32x4*>(src) + h);
      d.cw[4 * h] = v.x; d.cw[4 * h + 1] = v.y; d.cw[4 * h + 2] = v.z; d.cw[4 * h + 3] = v.w;
    }
  }
  if constexpr (CO < 3) d.pair = card_load<true>(reinterpret_cast<const uint32_t*>(card + in.off_meta[CO < 3 ? CO : 0]) + gsp / GS);
  return d;
}

template <int W>
__device__ __forceinline__ void decode_old(const OldSpan& d, uint32_t (&w)[16]) {
  uint32_t cw[W];
#pragma unroll
  for (int i = 0; i < W; ++i) cw[i] = d.cw[i];
  const float scale = half_bits_to_float(d.pair & 0xFFFFu), zero = half_bits_to_float(d.pair >> 16);
  if constexpr (W == 2) {
    decode_span<W>(cw, scale, zero, w);
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) decode_word<W>(cw[i], scale * 16777216.0f, zero, w + 16 / W * i);
  }
}

// Exchanges between the lanes l and l ^ 1: the odd lane's a becomes the even lane's b, and the other way round.
__device__ __forceinline__ void swap_between(uint32_t& a, uint32_t& b, bool odd) {
  const uint32_t from_a = dpp<kQuadXor1>(a), from_b = dpp<kQuadXor1>(b);
  a = odd ? from_b : a;
  b = odd ? b : from_a;
}

// Stores the N * 4 bytes of every lane at a place of its own.  Lane 2k + 1's place follows lane 2k's (a row has two spans at least), so
// they exchange every other sixteen bytes and each store writes 32 bytes in a row instead of 16 (32K tokens, 4 bits to 16: 1727 us and 1528;
// within fours of lanes and 64 bytes in a row 1187, but 8 registers more than eight waves a SIMD leave, which costs narrow rows more).
template <int N>
__device__ __forceinline__ void store_in_twos(uint8_t* dst, uint32_t (&w)[N], uint32_t lane) {
  const bool odd = (lane & 1u) != 0u;
#pragma unroll
  for (int j = 0; j < N; j += 8) {
#pragma unroll
    for (int k = j; k < j + 4; ++k) swap_between(w[k], w[k + 4], odd);
  }
  u32x4* d = reinterpret_cast<u32x4*>(dst - (odd ? N * 4 - 16 : 0));
#pragma unroll
  for (int j = 0; j < N; j += 8) {
    d[j / 4] = (u32x4){w[j], w[j + 1], w[j + 2], w[j + 3]};
    d[(N + j) / 4] = (u32x4){w[j + 4], w[j + 5], w[j + 6], w[j + 7]};
  }
}

// Stores the codes and the pair of span gsp of the outgoing class with width W.  Plain stores: the rows of a line may
// leave in different rounds, and the L2 puts the line together.
template <int W, int G>
__device__ __forceinline__ void store_span(uint8_t* card, const CardGeom& out, uint64_t gsp, uint32_t lane, bool live, uint32_t (&codes)[W], uint32_t pair) {
  constexpr int GS = G / 32, C = W == 2 ? 0 : W == 4 ? 1 : 2;
  if (!live) return;                                                   // both lanes of a pair are: they belong to one row
  uint8_t* dst = card + out.off_codes[C] + gsp * (4u * W);
  if constexpr (W == 2) *reinterpret_cast<u32x2*>(dst) = (u32x2){codes[0], codes[1]};
  if constexpr (W == 4) *reinterpret_cast<u32x4*>(dst) = (u32x4){codes[0], codes[1], codes[2], codes[3]};
  if constexpr (W == 8) store_in_twos<8>(dst, codes, lane);
  if ((lane & (GS - 1)) == 0) reinterpret_cast<uint32_t*>(card + out.off_meta[C])[gsp / GS] = pair;
}

template <int W, int G>
__device__ __forceinline__ void relabel_store(uint8_t* card, const CardGeom& out, uint32_t cw0, uint32_t cw1, uint32_t old_pair, uint64_t gsp,
                                              uint32_t lane, bool live) {
  uint32_t codes[W];
  const uint32_t cw[2] = {cw0, cw1};
  const uint32_t pair = relabel_span2<W, G / 32>(cw, old_pair, codes);
  store_span<W, G>(card, out, gsp, lane, live, codes, pair);
}

template <int W, int G>
__device__ __forceinline__ void quantize_store(uint8_t* card, const CardGeom& out, const uint32_t (&w)[16], uint64_t gsp, uint32_t lane, bool live) {
  uint32_t codes[W];
  const uint32_t pair = quantize_span<W, G / 32>(w, codes);            // every lane takes part: groups span lanes
  store_span<W, G>(card, out, gsp, lane, live, codes, pair);
}

// A round: up to 64 spans of rows list[first .. first + rows) of old class `co`.
struct Round {
  uint32_t co, first, rows;
};

struct Shared {
  u32x2 list[kWindow];                         // (slot in the incoming segment - across planes: row -, row of the window), sorted by old class
  uint32_t counts[kWindow / kWaveSize][8];
  uint32_t round_list[kMaxRounds];             // co | rows << 8 | first << 16
  uint32_t n_rounds;
};

// Window k of outgoing class C in the planes [p0, p1); across: window k of the class's rows of all planes.
template <int C, int G>
__device__ __forceinline__ void requant_window(const RequantArgs& a, const CardGeom& in, uint32_t k, bool across, uint32_t p0, uint32_t p1,
                                               Shared& sh) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const CardGeom& out = a.out;
  const uint32_t spr_shift = out.lpr_shift - 2u;                       // log2(spans per row)
  const uint32_t n_new = out.n[C];
  constexpr uint32_t kPer = kWindow / kBlockThreads;
  const uint32_t r0 = k * a.window;                                    // first row: of a plane, across planes of the segment
  const uint32_t rows = min(a.window, (across ? out.planes * n_new : n_new) - r0);

  // ---- look the rows up and sort them by old class
  uint32_t cls[kPer], slot[kPer], rank[kPer];                          // class 7: no row
  bool bad = false;
  {
    const uint32_t* order = reinterpret_cast<const uint32_t*>(a.card_out + out.off_order) + out.base[C];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t x = i * kBlockThreads + tid;
      cls[i] = 7u; slot[i] = 0u;
      if (x < rows) {
        cls[i] = 4u;
        uint32_t plane = 0, j = r0 + x;
        if (across) { plane = j / n_new; j -= plane * n_new; }
        const uint32_t t = order[j];
        if (t < out.tokens) {
          const uint32_t width = a.card_in[in.off_bits + t];
          const uint32_t sl = reinterpret_cast<const uint32_t*>(a.card_in + in.off_slot)[t];
          const uint32_t n_old = width == 2 ? in.n[0] : width == 4 ? in.n[1] : width == 8 ? in.n[2] : width == 16 ? in.n[3] : 0u;
          if (sl < n_old) { cls[i] = class_of(width); slot[i] = plane * n_old + sl; }
        }
        bad |= cls[i] == 4u;
      }
    }
  }
  if (bad && a.status) atomicOr(a.status, QKV_STATUS_BAD_ORDER);
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    uint64_t same = ~0ull;                                             // lanes with this lane's class
#pragma unroll
    for (uint32_t bit = 1; bit < 8u; bit <<= 1) {
      const uint64_t m = __builtin_amdgcn_ballot_w64((cls[i] & bit) != 0u);
      same &= (cls[i] & bit) ? m : ~m;
    }
    rank[i] = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    uint32_t* counts = sh.counts[i * kWavesPerBlock + wave];
    if (lane < 8u) counts[lane] = 0u;
    if (rank[i] == 0u) counts[cls[i]] = (uint32_t)__builtin_popcountll(same);
  }
  __syncthreads();
  uint32_t start = 0;                                                  // lane = class: its first place in the list
  {
    uint32_t total = 0, lower[kPer] = {};                              // of that class: in the window, in front of this wave's rows
#pragma unroll
    for (uint32_t w = 0; w < kPer * (uint32_t)kWavesPerBlock; ++w) {
      const uint32_t n = lane < kOld ? sh.counts[w][lane] : 0u;
      total += n;
#pragma unroll
      for (uint32_t i = 0; i < kPer; ++i) lower[i] += w < i * kWavesPerBlock + wave ? n : 0u;
    }
    start = wave_inclusive_scan(total) - total;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t at = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(cls[i] * 4u), (int)(start + lower[i])) + rank[i];
      if (cls[i] < kOld) sh.list[at] = (u32x2){slot[i], i * (uint32_t)kBlockThreads + tid};
    }
    if (wave == 0) {
      const uint32_t per_round = (uint32_t)kWaveSize >> spr_shift;     // rows
      const uint32_t rounds = (total + per_round - 1u) / per_round;
      const uint32_t inc = wave_inclusive_scan(rounds);
      if (lane == 63) sh.n_rounds = inc;
      for (uint32_t r = 0; r < rounds; ++r)
        sh.round_list[inc - rounds + r] = lane | (min(per_round, total - r * per_round) << 8) | ((start + r * per_round) << 16);
    }
  }
  __syncthreads();

  const uint32_t rounds = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.n_rounds);
  const uint32_t q = lane & ((1u << spr_shift) - 1u), row_of_lane = lane >> spr_shift;
  const auto round_at = [&](uint32_t r) {
    const uint32_t x = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.round_list[r]);
    const Round d = {x & 255u, x >> 16, (x >> 8) & 255u};
    return d;
  };
  const auto fetch = [&](const Round& d, uint32_t p, uint32_t in_row) {
    OldSpan o;
    if (d.co == 0u) o = fetch_old<0, G>(a.card_in, in, ((uint64_t)(p * in.n[0] + in_row) << spr_shift) + q);
    else if (d.co == 1u) o = fetch_old<1, G>(a.card_in, in, ((uint64_t)(p * in.n[1] + in_row) << spr_shift) + q);
    else if (d.co == 2u) o = fetch_old<2, G>(a.card_in, in, ((uint64_t)(p * in.n[2] + in_row) << spr_shift) + q);
    else if (d.co == 3u) o = fetch_old<3, G>(a.card_in, in, ((uint64_t)(p * in.n[3] + in_row) << spr_shift) + q);
    return o;
  };
  uint32_t p = p0, r = wave;
  while (r >= rounds) { r -= rounds; ++p; }
  if (p >= p1) return;
  Round next = round_at(r);
  u32x2 next_e = sh.list[next.first + min(row_of_lane, next.rows - 1u)];     // lanes past the round's rows repeat its last one
  OldSpan next_o = fetch(next, p, next_e.x);
  while (true) {
    const Round d = next;
    const u32x2 e = next_e;
    const OldSpan o = next_o;
    const uint32_t plane = p;
    r += kWavesPerBlock;
    while (r >= rounds) { r -= rounds; ++p; }
    const bool more = p < p1;
    if (more) {
      next = round_at(r);
      next_e = sh.list[next.first + min(row_of_lane, next.rows - 1u)];
      next_o = fetch(next, p, next_e.x);
    }
    const bool live = row_of_lane < d.rows;
    const uint64_t gsp = ((uint64_t)(plane * n_new + r0 + e.y) << spr_shift) + q;
    bool done = false;
    if constexpr (C < 3) {
      if (d.co == 0u && can_relabel(o.pair)) {
        relabel_store<(2 << C), G>(a.card_out, out, o.cw[0], o.cw[1], o.pair, gsp, lane, live);
        done = true;
      }
    }
    if (!done) {
      uint32_t w[16];
      if (d.co == 0u) decode_old<2>(o, w);
      else if (d.co == 1u) decode_old<4>(o, w);
      else if (d.co == 2u) decode_old<8>(o, w);
      else {
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = d.co == 3u ? o.cw[j] : 0u;
      }
      if constexpr (C < 3) {
        quantize_store<(2 << C), G>(a.card_out, out, w, gsp, lane, live);
      } else if (live) {
        store_in_twos<16>(a.card_out + out.off_fp16 + gsp * 64u, w, lane);
      }
    }
    if (!more) break;
  }
}

template <int G>
__global__ __launch_bounds__(kBlockThreads) void requant_kernel(RequantArgs a) {
  __shared__ Shared sh;
  CardGeom in;
  if (!card_geometry_from_header(a.card_in, a.card_in_bytes, a.layers, a.kv_heads, a.head_dim, a.group_size, a.tokens, in))
    return;                                   // uniform over the grid
  uint32_t k = blockIdx.y * gridDim.x + blockIdx.x;
  if (k >= a.blocks) return;
  const bool across = a.group_planes == 0u;
  uint32_t p0 = 0, p1 = 1u;
  if (!across) {
    const uint32_t group = k / a.stride;
    k -= group * a.stride;
    if (k >= a.windows[0] + a.windows[1] + a.windows[2] + a.windows[3]) return;
    p0 = group * a.group_planes;
    p1 = min(p0 + a.group_planes, a.out.planes);
  }
  if (k < a.windows[0]) requant_window<0, G>(a, in, k, across, p0, p1, sh);
  else if ((k -= a.windows[0]) < a.windows[1]) requant_window<1, G>(a, in, k, across, p0, p1, sh);
  else if ((k -= a.windows[1]) < a.windows[2]) requant_window<2, G>(a, in, k, across, p0, p1, sh);
  else requant_window<3, G>(a, in, k - a.windows[2], across, p0, p1, sh);
}


// ---- long cards of narrow rows ----

// A span as it lies in the incoming card, for the kernel below: its codes (or its 32 raw values) and its pair.  2-bit codes are the first
// half of c[0]; behind them are whatever bytes follow in the card.
struct WideSpan {
  u32x4 c[4];
  uint32_t pair;
};
typedef u32x4 __attribute__((aligned(8))) u32x4_a8;

template <int W>
__device__ __forceinline__ void decode_wide(const WideSpan& d, uint32_t (&w)[16]) {
  OldSpan o;
#pragma unroll
  for (int i = 0; i < W; ++i) o.cw[i] = d.c[i / 4][i % 4];
  o.pair = d.pair;
  decode_old<W>(o, w);
}

constexpr uint32_t kTokenThreads = 512, kTokenWaves = kTokenThreads / kWaveSize;
constexpr uint32_t kTokenRows = kTokenThreads;   // rows (plane, token) that a workgroup looks up and sorts: one a thread
constexpr uint32_t kPairs = 20;               // pairs of an old class - 0 .. 3, and 4: not placed by the incoming tables - and a new one
constexpr uint32_t kNoRow = 31;

struct TokenArgs {
  const uint8_t* card_in;
  uint64_t card_in_bytes;
  uint32_t layers, kv_heads, head_dim, group_size;
  uint64_t tokens;
  CardGeom out;                 // the outgoing card's geometry (host-known counts)
  uint8_t* card_out;
  uint32_t* status;             // may be null; holds the verdict on the incoming header already (classify_kernel)
  uint32_t rows;                // planes / group_planes * tokens
  uint32_t group_planes;        // planes that a workgroup does one after the other, with one look-up and sort
};

struct TokenShared {
  static constexpr uint32_t kRounds = kTokenRows * 8u / kWaveSize + kPairs;      // 8 spans a row at most
  u32x2 list[kTokenRows];                           // row of the old class's segment, row of the new one's; sorted by pair of classes
  uint32_t counts[kTokenWaves][32];
  uint32_t found[kRounds];                     // rounds: pair | rows << 8 | first place in the list << 16
  u32x4 place[kRounds / 4 + 1];                // where in the window a round's middle row is << 12 | its number
  uint32_t rounds[kRounds];                    // the same as found, by place
  u32x4 sections[8];                           // where the codes and the pairs of an old class begin
  uint32_t n_old[8];
};

template <int G>
__global__ __launch_bounds__(kTokenThreads) void requant_tokens_kernel(TokenArgs a) {
  __shared__ TokenShared sh;
  CardGeom in;
  if (!card_geometry_from_header(a.card_in, a.card_in_bytes, a.layers, a.kv_heads, a.head_dim, a.group_size, a.tokens, in))
    return;                                   // uniform over the grid
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const CardGeom& out = a.out;
  const uint32_t spr_shift = out.lpr_shift - 2u;                       // log2(spans per row)
  const uint32_t T = out.tokens;

  if (tid == 0) {                             // a choice among the members of `in` would be loaded from scratch memory, by index
    const auto at = [](uint64_t codes, uint64_t pairs) {
      return (u32x4){(uint32_t)codes, (uint32_t)(codes >> 32), (uint32_t)pairs, (uint32_t)(pairs >> 32)};
    };
#pragma unroll
    for (int c = 0; c < 3; ++c) sh.sections[c] = at(in.off_codes[c], in.off_meta[c]);
    sh.sections[3] = at(in.off_fp16, in.off_fp16);
    sh.sections[4] = at(0u, 0u);
#pragma unroll
    for (int c = 0; c < 4; ++c) sh.n_old[c] = in.n[c];
    sh.n_old[4] = 0u;
  }

  // ---- look the rows up and sort them by pair of classes
  uint32_t pair_of = kNoRow, rank;
  u32x2 entry = {};
  {
    // Workgroups are dealt out strictly in turn, to the eight XCDs and to the parts of each: where a plane's windows are a multiple
    // of that, the same tokens of all planes meet on the same compute units, and where widths go with the tokens some have all of the
    // wide rows (16384 tokens sorted by width, 6 to 4: 511 us, with every 64 workgroups in an order of their own 343).
    uint32_t window = blockIdx.x;
    if ((window | 63u) < gridDim.x) window = (window & ~63u) | ((window * 21u + (window >> 6) * 13u) & 63u);
    const uint32_t r0 = window * kTokenRows, rows = min(kTokenRows, a.rows - r0);
    const uint32_t group0 = r0 / T, t0 = r0 - group0 * T;
    const bool as_counted = (reinterpret_cast<const uint32_t*>(a.card_out)[48] & QKV_STATUS_BAD_COUNTS) == 0u;
    bool bad = false;
    if (tid < rows) {
      uint32_t group = 0, t = t0 + tid;
      if (T >= kTokenRows) { if (t >= T) { group = 1u; t -= T; } }
      else { group = t / T; t -= group * T; }
      const uint32_t plane = (group0 + group) * a.group_planes;
      uint32_t cn, sn;
      if (as_counted) {
        cn = class_of(a.card_out[out.off_bits + t]);
        sn = reinterpret_cast<const uint32_t*>(a.card_out + out.off_slot)[t];
      } else {                                                         // rows as the caller's counts say, tokens as order[] says
        cn = t < out.base[1] ? 0u : t < out.base[2] ? 1u : t < out.base[3] ? 2u : 3u;
        sn = t - (cn == 0u ? out.base[0] : cn == 1u ? out.base[1] : cn == 2u ? out.base[2] : out.base[3]);
        t = min(reinterpret_cast<const uint32_t*>(a.card_out + out.off_order)[t], T - 1u);
      }
      const uint32_t n_new = cn == 0u ? out.n[0] : cn == 1u ? out.n[1] : cn == 2u ? out.n[2] : out.n[3];
      const uint32_t width = a.card_in[in.off_bits + t];
      const uint32_t so = reinterpret_cast<const uint32_t*>(a.card_in + in.off_slot)[t];
      const uint32_t n_old = width == 2 ? in.n[0] : width == 4 ? in.n[1] : width == 8 ? in.n[2] : width == 16 ? in.n[3] : 0u;
      const uint32_t co = so < n_old ? class_of(width) : 4u;
      bad = co == 4u;
      if (sn < n_new) pair_of = co * 4u + cn;
      entry = (u32x2){plane * n_old + so, plane * n_new + sn};
    }
    if (bad && a.status) atomicOr(a.status, QKV_STATUS_BAD_ORDER);
    uint64_t same = ~0ull;                                             // lanes with this lane's pair
#pragma unroll
    for (uint32_t bit = 1; bit < 32u; bit <<= 1) {
      const uint64_t m = __builtin_amdgcn_ballot_w64((pair_of & bit) != 0u);
      same &= (pair_of & bit) ? m : ~m;
    }
    rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    if (lane < 32u) sh.counts[wave][lane] = 0u;
    if (rank == 0u) sh.counts[wave][pair_of] = (uint32_t)__builtin_popcountll(same);
  }
  __syncthreads();
  const uint32_t per_shift = 6u - spr_shift, per_round = 1u << per_shift;     // rows of a round
  uint32_t n_rounds;
  {
    uint32_t total = 0, lower = 0;                                     // lane = pair: its rows in the window, and in front of this wave's
#pragma unroll
    for (uint32_t w = 0; w < kTokenWaves; ++w) {
      const uint32_t n = lane < kPairs ? sh.counts[w][lane] : 0u;
      total += n;
      lower += w < wave ? n : 0u;
    }
    const uint32_t start = wave_inclusive_scan(total) - total;         // first place in the list
    const uint32_t own = (total + per_round - 1u) >> per_shift;
    const uint32_t inc = wave_inclusive_scan(own);
    n_rounds = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    if (wave == 0 && lane < 4u) reinterpret_cast<uint32_t*>(sh.place)[n_rounds + lane] = ~0u;
    const int from = (int)(pair_of * 4u);
    const uint32_t first = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)start);
    const uint32_t rel = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)lower) + rank;
    const uint32_t info = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)((inc - own) | (total << 16)));
    if (pair_of < kPairs) {
      const uint32_t begin = rel & ~(per_round - 1u), rows = min(per_round, (info >> 16) - begin);
      sh.list[first + rel] = entry;
      if (rel == begin + rows / 2u) {
        const uint32_t r = (info & 0xFFFFu) + (rel >> per_shift);
        sh.found[r] = pair_of | (rows << 8) | ((first + begin) << 16);
        reinterpret_cast<uint32_t*>(sh.place)[r] = (tid << 12) | r;
      }
    }
  }
  __syncthreads();
  if (tid < n_rounds) {
    const uint32_t mine = reinterpret_cast<const uint32_t*>(sh.place)[tid];
    uint32_t before = 0;
    for (uint32_t j = 0; j < (n_rounds + 3u) / 4u; ++j) {
      const u32x4 p = sh.place[j];
      before += (uint32_t)(p.x < mine) + (uint32_t)(p.y < mine) + (uint32_t)(p.z < mine) + (uint32_t)(p.w < mine);
    }
    sh.rounds[before] = sh.found[tid];
  }
  __syncthreads();
  if (n_rounds == 0u) return;                                          // only where the caller's counts are wrong

  const uint32_t q = lane & ((1u << spr_shift) - 1u), row_of_lane = lane >> spr_shift;
  uint32_t r = wave, p = 0;
  while (r >= n_rounds) { r -= n_rounds; ++p; }
  if (p >= a.group_planes) return;
  uint32_t d, row_out;
  WideSpan o = {};
  const auto fetch = [&]() {
    d = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.rounds[r]);
    const u32x2 e = sh.list[(d >> 16) + min(row_of_lane, ((d >> 8) & 255u) - 1u)];   // lanes past the round's rows repeat its last one
    const uint32_t co = (d >> 2) & 7u, cn = d & 3u;
    row_out = e.y + p * (cn == 0u ? out.n[0] : cn == 1u ? out.n[1] : cn == 2u ? out.n[2] : out.n[3]);
    // One sequence of loads for all classes, each into registers of its own: out of branches that load into the same ones they
    // came with copies behind each, and waits in front of the copies.  Raw rows have no pair and load their own start in its place; rows
    // that the incoming tables don't place load the card's.
    const uint64_t gsp = co < 4u ? ((uint64_t)(e.x + p * sh.n_old[co]) << spr_shift) + q : 0u;
    const u32x4 at = sh.sections[co];
    const uint64_t codes = (uint64_t)at.x | (uint64_t)at.y << 32, meta = (uint64_t)at.z | (uint64_t)at.w << 32;
    const uint8_t* src = a.card_in + codes + (gsp << (3u + co));
    o.c[0] = *reinterpret_cast<const u32x4_a8*>(src);
    o.pair = *reinterpret_cast<const uint32_t*>(co < 3u ? a.card_in + meta + gsp / (G / 32) * 4u : src);
    if (co >= 2u) o.c[1] = reinterpret_cast<const u32x4*>(src)[1];
    if (co == 3u) {
      o.c[2] = reinterpret_cast<const u32x4*>(src)[2];
      o.c[3] = reinterpret_cast<const u32x4*>(src)[3];
    }
  };
  fetch();
  while (true) {
    const uint32_t co = (d >> 2) & 7u, cn = d & 3u;
    const bool live = row_of_lane < ((d >> 8) & 255u);
    const uint64_t gsp = ((uint64_t)row_out << spr_shift) + q;
    const bool relabel = co == 0u && cn != 3u && can_relabel(o.pair);
    uint32_t w[16];
    if (relabel) { w[0] = o.c[0].x; w[1] = o.c[0].y; w[2] = o.pair; }
    else if (co == 0u) decode_wide<2>(o, w);
    else if (co == 1u) decode_wide<4>(o, w);
    else if (co == 2u) decode_wide<8>(o, w);
    else {
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = co == 3u ? o.c[j / 4][j % 4] : 0u;
    }
    // The next round's loads go to the registers that this round's came to, once it is decoded: copies of them, with the loads
    // in front of the decoding, were a fifth of the loop's vector instructions.
    r += kTokenWaves;
    while (r >= n_rounds) { r -= n_rounds; ++p; }
    const bool more = p < a.group_planes;
    if (more) fetch();
    if (relabel) {
      if (cn == 0u) relabel_store<2, G>(a.card_out, out, w[0], w[1], w[2], gsp, lane, live);
      else if (cn == 1u) relabel_store<4, G>(a.card_out, out, w[0], w[1], w[2], gsp, lane, live);
      else relabel_store<8, G>(a.card_out, out, w[0], w[1], w[2], gsp, lane, live);
    }
    else if (cn == 0u) quantize_store<2, G>(a.card_out, out, w, gsp, lane, live);
    else if (cn == 1u) quantize_store<4, G>(a.card_out, out, w, gsp, lane, live);
    else if (cn == 2u) quantize_store<8, G>(a.card_out, out, w, gsp, lane, live);
    else if (live) store_in_twos<16>(a.card_out + out.off_fp16 + gsp * 64u, w, lane);
    if (!more) break;
  }
}

}  // namespace

hipError_t launch_requant(const uint8_t* card_in, uint64_t card_in_bytes, const CardGeom& out, uint8_t* card_out,
                          uint32_t* status, hipStream_t stream) {
  RequantArgs a;
  a.card_in = card_in;
  a.card_in_bytes = card_in_bytes;
  a.layers = out.layers; a.kv_heads = out.kv_heads; a.head_dim = out.head_dim; a.group_size = out.group_size;
  a.tokens = out.tokens;
  a.out = out;
  a.card_out = card_out;
  a.status = status;
  // Windows of a plane end where its rows of the width end, and each is sorted and cut into rounds by itself: with a few
  // hundred tokens most rounds are then partly empty.  Short cards' windows run across planes instead, every one
  // full, at the price of a division per row and of a plane's widths being read at different times, which costs more
  // the less of the cards the 256 MB memory-side cache holds.  Where windows of a plane would be fewer than fill the
  // chip, longer cards' run across planes too.  Of the shapes that come here, whole call with the classification, us, with windows of a plane
  // and across planes: 512 planes of 128 values, 200 tokens, budget 3 to 2.5, 19.9 and 13.9; 500 26.3 and 19.2; 1000 31.0 and 26.2;
  // 1400, 6 to 4, 40.7 and 40.1; 1900 50.9 and 51.1; wide rows, 4000 tokens, 5 to 8 142 and 159, 9.5 to 6.5 148 and 155, 8 bits to 8 126 and 118.  512 planes of
  // 64 values, 1500 tokens, 3 to 2.5 31.5 and 26.8, 1800 34.5 and 30.2, 6 to 4 33.6 and 32.6, 4000 57.9 and 58.6, 8192 124 and 130.  1024
  // planes of 256 values, 9.5 to 6.5, 400 tokens 47.6 and 49.0, 900 131 and 139.  64 planes of 6000 tokens of 128 values 24.4 and 22.7, 16 of 32768
  // 29.9 and 29.5.  Smaller windows while there are few (kernel alone): 200 tokens, 6 to 4, 11.6 with 128 rows and 12.1 with 256, 64 tokens 7.4
  // with 64 rows and 8.0 with 128.
  const uint64_t rows = (uint64_t)out.planes * out.tokens;
  const uint64_t values = rows * out.head_dim;
  // Long cards: the windows of tokens, unless a head has 64 dimensions (windows of half the bytes, and as many rounds that are not
  // full) or rows are wide (whole lines that nobody else reads: nothing to gain, and more to lose where widths are sorted along the tokens, as
  // they nearly are where scores follow the position).  Whole call, us, with windows of a width and of tokens:
  // 512 planes of 128 values, 1500 tokens, 3 to 2.5 33.7 and 35.3, 2000 43.4 and 41.8, 6 to 4 62.4 and 59.7, 16000 410 and 371;
  // 256 planes of 256 values, 1500 tokens, 6 to 4 46.6 and 46.2, 2000 58.9 and 57.2, 16000 395 and 356; 512 of 64, 5000 tokens, 6 to 4
  // 85.1 and 85.9, 16000, 8 to 5, 253 and 267; 512 of 128, 16384 tokens, 16 to 4 541 and 567, 8 to 8 568 and 588, 8 to 6 511 and 498,
  // 9.5 to 6.5 550 and 551, sorted 9 to 6 433 and 463, 6 to 4 328 and 347, 3 to 2.5 224 and 227.
  // The incoming card's length is all that is known here of its widths: in a longer buffer it counts as a card of wider rows.
  const uint64_t bytes = card_in_bytes + out.total;
  if (out.head_dim >= 128u && values >= 131072000ull && 2u * card_in_bytes <= 3u * values && out.total <= values && bytes <= 2u * values) {
    TokenArgs t;
    t.card_in = card_in; t.card_in_bytes = card_in_bytes;
    t.layers = out.layers; t.kv_heads = out.kv_heads; t.head_dim = out.head_dim; t.group_size = out.group_size;
    t.tokens = out.tokens;
    t.out = out;
    t.card_out = card_out;
    t.status = status;
    // Two planes with one look-up and sort where rows are narrow and the look-ups' share is large; wider ones want the planes that are worked on at a
    // time to be neighbours, unless the cards sit in the memory-side cache.  A row of 256 values has fewer look-ups a byte, and there the chip must
    // stay full with half the workgroups.  Both cards' bits a value decide (one plane and two, us; 2 to 2 bits 16384 tokens 215 and 175, 3 to 2.5
    // 8192 151 and 136, 16384 291 and 255, 4 to 2 294 and 265, 5 to 2.5 8192 166 and 161; 6 to 4 2001 tokens 47.3 and 49.1, 8192 197 and 211, 8 to
    // 5 235 and 256, 8 bits to 4 3000 72.1 and 77.1, 32768, 6 to 4, 745 and 790; between them 5 to 3 8192 170 and 174, 4 to 4 176 and 185, but 2001 44.8
    // and 43.9; all of 4 bits to 4 again 8192 163 and 149, 16384 317 and 285.  256 values, 3 to 2.5: 2001 tokens 36.3 and 38.4, 6000 91.6 and
    // 90.0, 8192 123 and 118, 4 to 3 6000 103 and 106).
    // A card has an even number of planes, and a grid fewer than 2^32 threads.
    const bool one_width = out.n[0] == out.tokens || out.n[1] == out.tokens || out.n[2] == out.tokens || out.n[3] == out.tokens;
    const bool two = out.head_dim > 128u ? 16u * bytes <= 15u * values && rows >= 2u * 1024u * kTokenRows
                                         : 16u * bytes <= 19u * values || (one_width && card_in_bytes <= out.total) ||
                                           (16u * bytes <= 21u * values && bytes <= (256ull << 20));
    t.group_planes = two || rows >= (1ull << 31) ? 2u : 1u;
    t.rows = out.planes / t.group_planes * out.tokens;
    const dim3 grid((t.rows + kTokenRows - 1u) / kTokenRows), block(kTokenThreads);
    switch (out.group_size) {
      case 32: hipLaunchKernelGGL(requant_tokens_kernel<32>, grid, block, 0, stream, t); break;
      case 64: hipLaunchKernelGGL(requant_tokens_kernel<64>, grid, block, 0, stream, t); break;
      default: hipLaunchKernelGGL(requant_tokens_kernel<128>, grid, block, 0, stream, t); break;
    }
    return hipGetLastError();
  }
  const bool cached = card_in_bytes + out.total <= (192ull << 20);
  const bool across = rows < 1536u * kWindow || (cached ? out.tokens < 1536u : (uint64_t)out.tokens * out.head_dim < 900u * 128u);
  a.window = !across || rows > 512u * kWindow ? kWindow : rows > 128u * kWindow ? kWindow / 2u : kWindow / 4u;
  uint64_t blocks = 0;
  for (int c = 0; c < 4; ++c) {
    a.windows[c] = (uint32_t)(((across ? (uint64_t)out.planes : 1ull) * out.n[c] + a.window - 1u) / a.window);
    blocks += a.windows[c];
  }
  a.group_planes = 0u;
  a.stride = 1u;
  if (!across) {
    // A workgroup's look-ups are worth sharing between planes while the chip stays full several times over and both cards
    // sit in the memory-side cache (512 planes of 64 values, 8192 tokens, 3 to 2.5: 76.1 us with two planes, 94.3 with one, 6 to 4 124 and 127, but 8 to 5
    // 144 and 136; 20000 tokens, 3 to 2.5, 200 and 245); larger cards of wide rows want a plane's windows, which share lines of the
    // incoming card, to run at the same time (60000 tokens, 8 to 5: 950 us with two planes, 898 with one; 512 of 128 values, 8192
    // tokens, 9.5 to 6.5, 309 and 285).
    const bool resident = out.total <= kCacheResidentCardBytes && card_in_bytes <= kCacheResidentCardBytes;
    uint32_t group = resident ? kMaxPlanes : 1u;
    while (group > 1u && blocks * ((out.planes + group - 1u) / group) < 8192u) group /= 2u;
    a.group_planes = group;
    // Workgroups go to the eight XCDs in turn: with eight windows a plane, or a multiple, a width's windows of all planes would
    // meet on the same ones (1500 tokens, 8 windows: 45.6 us, with a ninth workgroup that leaves at once 37.1).  Windows of
    // one width are all alike and need none (2000 tokens, 8 bits to 2: 44.6 us without, 46.1 with).
    const bool one_width = blocks == a.windows[0] || blocks == a.windows[1] || blocks == a.windows[2] || blocks == a.windows[3];
    a.stride = (uint32_t)blocks | (one_width ? 0u : 1u);
    blocks = (uint64_t)a.stride * ((out.planes + group - 1u) / group);
  }
  a.blocks = (uint32_t)blocks;
  const uint32_t grid_y = (a.blocks + kMaxGridX - 1u) / kMaxGridX, grid_x = (a.blocks + grid_y - 1u) / grid_y;
  const dim3 grid(grid_x, grid_y), block(kBlockThreads);
  switch (out.group_size) {
    case 32: hipLaunchKernelGGL(requant_kernel<32>, grid, block, 0, stream, a); break;
    case 64: hipLaunchKernelGGL(requant_kernel<64>, grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL(requant_kernel<128>, grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace qkv
