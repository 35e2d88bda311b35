// attend.hip — decode-step attention of one new query token directly over a card (paper
// Sec. 4.3: consuming a foreign quantized cache inside attention instead of rebuilding the
// dense fp16 cache first, which the paper leaves as future work).
//
// For every layer l and query head hq (kv head h = hq / R, R = query heads per kv head):
//     s_t = scale * <q[l,hq], K^[l,h,t]>,   o = softmax(s) . V^[l,h,:],   lse = log sum exp s
// with K^, V^ the dequantized fp16 values, exactly those the injection kernel would write.
// A softmax sum does not care about the order of its terms, so the card's segments are used
// as they lie: no order[] lookup, no gather.
//
// Work decomposition.  A task is up to `chunk` consecutive rows of one width's
// segment for one (layer, kv head), for all R query heads.  A wave takes every a.waves-th task of a pair and leaves an unnormalised
// partial (running maximum m, sum l, sum of p.V^) in a workspace, where it finds the sums of p.V^ again after its next task; a second
// kernel merges the partials of each (layer, query head).  Inside a task, in rounds of 2048 values (16 tokens of 128 dimensions, 32 of 64):
//   scores   a lane reads a span of 32 codes and its pair, decodes it to four MFMA operands of 8 dimensions,
//            and four MFMAs accumulate q.K^ for the round's tokens and the kv head's query
//            heads (the k index of the MFMA is a fixed permutation of the head dimension,
//            applied to q and K^ alike).  Scores go to LDS.
//   softmax  one maximum per head over the task's tokens, p = exp2(s - m) back into LDS, as an fp16 high part and
//            the fp16 remainder.
//   values   the round's packed V rows are regrouped through LDS (still packed; raw rows are read as they are wanted) so
//            that a lane holds 4 tokens x 8 dimensions (64 dimensions: 8 x 4), decodes them into MFMA operands of 4 tokens
//            x 2 dimensions, and MFMAs add p.V^.
// Both products are v_mfma_f32_16x16x32_f16 (see attend_task).  head_dim 256 is two slabs of 128.
// 2-bit spans, most of a card at low budgets, are not decoded by arithmetic: a group has only
// four decoded values, which are computed once and picked by v_perm_b32.  Rounds are taken in whole groups of 4 / 3 / 2 /
// 1 (at 2 / 4 / 8 / 16 bits; 64 and 256 dimensions: 2 / 2 / 1 / 1) without a branch in between; rounds past a task's end see zeros and
// count as -inf.  96 .. 127 registers and 9.5 KiB of LDS per wave: four waves per SIMD.
//
// Vector instructions of a round of 16 tokens x 128 dimensions with up to 4 query heads, at 2 / 4 / 8 bits: scores 61 / 85 / 80, softmax 10,
// values 38 / 91 / 88, and 8 MFMAs of 16 cycles; at 2 bits the vector pipes are then about 70 % and LDS, most of it the value
// pass's look-ups, 65 % busy.  With v_mfma_f32_4x4x4_16b_f16, whose operands are four tokens of one dimension,
// values had to be turned from pairs of dimensions into pairs of tokens, sums added up across lanes, high and low parts of
// the weights took an MFMA each: 84, 18 and 112 at 2 bits, 24 MFMAs of 8 cycles.  Whole call, 32 query heads on 8 kv heads, 32
// layers, us, then and now (with cut_tasks; card not in cache): 8192 tokens at budget 3 80 and 65, all 2 bits 67 and 57, 4 bits 85 and 78,
// 8 bits 124.6 and 122.5; 1024 tokens at budget 5 20.9 and 17.7.  64 dimensions had left half the lanes idle, and more than 4 heads
// took the 16 x 16 x 16 product: 8 heads, 3877 tokens of 128 pairs 30.1 and 20.3; 16 heads of 256 dimensions, 22950 tokens of 64 pairs 331 and 265.

#include <algorithm>
#include <atomic>
#include <cmath>

#include "attend_cut.h"
#include "qkv_common.h"
#include "qkv_decode.h"

namespace qkv {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct AttendArgs {
  const uint8_t* card;
  uint64_t card_bytes;
  uint32_t layers, kv_heads, head_dim, group_size;
  uint64_t tokens;
  const uint16_t* q;       // fp16 [L][Hq][D]
  uint32_t q_heads;        // Hq
  uint32_t rep;            // R = Hq / H, 1 .. 16
  float scale_log2;        // softmax scale times log2(e); its absolute value where keys are not grouped per channel, and then
  uint32_t q_flip;         // the sign bits to turn in q for the scale's own: the largest score is the one of the largest product
  float* part_o;           // [L*H][waves][R][D] unnormalised sums of p.V^
  float* part_ml;          // [L*H][waves][R][2]  (m in log2 units, l)
  uint32_t chunk, rows;    // tokens per task at most: what the scores' LDS holds, and in one turn (see cut_tasks)
  uint32_t waves;          // per (layer, kv head); the workspace has room for a partial each
  uint32_t flat;           // the grid is one row
  uint32_t unit[4];        // tokens of a class that make up one unit (read where keys are grouped per channel, kUnit otherwise)
  uint32_t fit[4], fit_rows[4];      // chunk / unit, rows / unit
  float* out;              // fp32 [L][Hq][D]
  float* lse;              // fp32 [L][Hq] or null
  uint32_t* status;        // or null
  uint32_t* valid;         // one word of the workspace: the partials of every pair that are to be merged, 0 when the header was refused
};

// What a lane holds of one round's rows before it is decoded: the codes of a span of 32 values (or raw values) and its pair.
template <int W, int G>
struct SpanData {
  uint32_t cw[W == 16 ? 16 : W];
  uint32_t pair;
};

// A task's rows of one plane as two buffers that end with the task's last row: what is read past them is zero, in
// hardware, so no round needs a test, a mask or zeros of its own.  `codes_at` and `pairs_at` are the lane's own
// offsets in round 0; every round is a fixed number of bytes further.
struct RowStream {
  __amdgpu_buffer_rsrc_t codes, pairs;
  uint32_t codes_at, pairs_at;
};

__device__ inline uint64_t uniform64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// The untyped buffer [at, at + bytes): a load that would reach past its end gives zero.
__device__ inline __amdgpu_buffer_rsrc_t bounded(const uint8_t* at, uint32_t bytes) {
  const uint64_t p = uniform64(reinterpret_cast<uint64_t>(at));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(p), 0, (int)(uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00027000);
}

// Rows of a round, and how lane (n, kq) = (lane % 16, lane / 16) sits in it.  A round is 2048 values of a slab of up to 128
// dimensions: 16 tokens, or 32 where a token has 64 dimensions.
template <int DS> struct RoundGeo {
  static constexpr uint32_t kTokens = DS == 2 ? 32u : 16u;
  static constexpr uint32_t kSpans = DS == 2 ? 2u : 4u;                // spans of a token in the slab
  // loader side: the lane's row of the round and its span of that row
  static __device__ inline uint32_t row(uint32_t n, uint32_t kq) { return DS == 2 ? n + 16u * (kq >> 1) : n; }
  static __device__ inline uint32_t span(uint32_t kq) { return DS == 2 ? (kq & 1u) : kq; }
};

template <int W, int DS> struct RowBytes {
  static constexpr uint32_t kCodes = (uint32_t)DS * 4u * W;            // of a row; raw rows: 64 bytes per span
};

// The rows [row0, row0 + cnt) of class c, read from span `span` of row `row` of every round.
template <int W, int G, int DS>
__device__ inline RowStream row_stream(const uint8_t* card, const CardGeom& g, int c, uint64_t row0, uint32_t cnt, uint32_t row, uint32_t span) {
  constexpr uint32_t kPairBytes = (uint32_t)DS * 32u / G * 4u;
  RowStream s;
  const uint64_t off = W == 16 ? g.off_fp16 : g.off_codes[c];
  s.codes = bounded(card + off + row0 * RowBytes<W, DS>::kCodes, cnt * RowBytes<W, DS>::kCodes);
  s.codes_at = row * RowBytes<W, DS>::kCodes + span * (4u * W);
  if constexpr (W != 16) {
    s.pairs = bounded(card + g.off_meta[c] + row0 * kPairBytes, cnt * kPairBytes);
    s.pairs_at = row * kPairBytes + span / (G / 32u) * 4u;
  } else {
    s.pairs = s.codes;
    s.pairs_at = 0u;
  }
  return s;
}

__device__ inline u32x4 buffer_load4(__amdgpu_buffer_rsrc_t r, uint32_t at) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0));
}
__device__ inline u32x2 buffer_load2(__amdgpu_buffer_rsrc_t r, uint32_t at) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)at, 0, 0));
}

// Issues the loads of the lane's span in round rd; nothing is decoded yet.  Zeros past the task's last row.
template <int W, int G, int DS>
__device__ inline SpanData<W, G> fetch_span(const RowStream& s, uint32_t rd) {
  constexpr uint32_t kRows = RoundGeo<DS>::kTokens;
  SpanData<W, G> d;
  const uint32_t at = s.codes_at + rd * (kRows * RowBytes<W, DS>::kCodes);
  if constexpr (W == 2) {
    const u32x2 t = buffer_load2(s.codes, at);
    d.cw[0] = t.x; d.cw[1] = t.y;
  } else {
#pragma unroll
    for (int h = 0; h < W / 4; ++h) {
      const u32x4 t = buffer_load4(s.codes, at + 16u * h);
      d.cw[4 * h] = t.x; d.cw[4 * h + 1] = t.y; d.cw[4 * h + 2] = t.z; d.cw[4 * h + 3] = t.w;
    }
  }
  d.pair = 0u;
  if constexpr (W != 16) d.pair = __builtin_amdgcn_raw_buffer_load_b32(s.pairs, (int)(s.pairs_at + rd * (kRows * ((uint32_t)DS * 32u / G * 4u))), 0, 0);
  return d;
}

// The 32 values of a fetched span as 16 packed fp16 pairs (2 bits: see decode_fetched_bytes).
template <int W, int G>
__device__ inline void decode_fetched(const SpanData<W, G>& d, uint32_t (&out)[16]) {
  if constexpr (W == 16) {
#pragma unroll
    for (int i = 0; i < 16; ++i) out[i] = d.cw[i];
  } else {
    const float s = half_bits_to_float(d.pair & 0xFFFFu) * 16777216.0f;
    const float z = half_bits_to_float(d.pair >> 16);
#pragma unroll
    for (int i = 0; i < W; ++i) decode_word<W>(d.cw[i], s, z, out + 16 / W * i);
  }
}

// The 32 values of a 2-bit span by byte selection: the low bytes of the span's four values and their high bytes are picked
// apart, four codes at a time, and put together: out[8 w + 2 k + h] = values 16 w + 8 h + k and 16 w + 8 h + 4 + k.
// 1.8 vector instructions a value where the selector table in LDS takes 0.75 and a look-up for every four values, but the
// look-ups' bank conflicts filled the LDS pipe while the vector units had room (8K tokens of 2 bits 56.6 -> 53.6 us).
template <int G>
__device__ inline void decode_fetched_bytes(const SpanData<2, G>& d, uint32_t (&out)[16]) {
  const float s = half_bits_to_float(d.pair & 0xFFFFu), z = half_bits_to_float(d.pair >> 16);
  const uint32_t x01 = decode_pair(0.0f, 1.0f, s, z), x23 = decode_pair(2.0f, 3.0f, s, z);
  const uint32_t low = __builtin_amdgcn_perm(x23, x01, 0x06040200u), high = __builtin_amdgcn_perm(x23, x01, 0x07050301u);
#pragma unroll
  for (int w = 0; w < 2; ++w) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t code = (d.cw[w] >> (2 * k)) & 0x03030303u;            // codes k, 4 + k, 8 + k, 12 + k of the word
      const uint32_t lo = __builtin_amdgcn_perm(low, low, code), hi = __builtin_amdgcn_perm(high, high, code);
      out[8 * w + 2 * k] = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
      out[8 * w + 2 * k + 1] = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
    }
  }
}

// The 32 values of q that meet such a span, in the same order.
__device__ inline void order_q2(u32x4 (&raw)[4]) {
  uint32_t out[16];
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int first = 8 * (x >> 3) + 4 * (x & 1) + ((x >> 2) & 1);         // the word of value 16 w + 8 h + k, and k's lowest bit
    out[x] = __builtin_amdgcn_perm(raw[(first + 2) >> 2][(first + 2) & 3], raw[first >> 2][first & 3], ((x >> 1) & 1) ? 0x07060302u : 0x05040100u);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) raw[j] = (u32x4){out[4 * j], out[4 * j + 1], out[4 * j + 2], out[4 * j + 3]};
}

// ---- the LDS tile of a round: packed rows, regrouped ---------------------------------------------
//
// Used for the value rows (2, 4 and 8 bits) of every card and for the key rows of cards grouped per channel.  In both
// cases the MFMA contracts over the tile's rows, so a lane must hold several rows of the same columns; the loader lane holds
// one span of one row.  The rows are dropped into LDS still packed and picked up again in pieces; only codes
// cross LDS, never decoded values.

// Rows of 16 spans, or 32 of 8 bytes at head_dim 64.  The pitch keeps the rows that a read instruction touches (4 apart) on
// different banks and every span where its store of 8 (2 bits) or 16 bytes may lie (4 bits, 64 dimensions: 48 bytes; with 40, every odd
// row's store 8 bytes off, 16 shapes took 1.6 % longer).  Behind the rows, as [span][row]: the 64 pairs as two floats (2-bit rows: 64 four-value tables), and
// at 2 bits the 2 KiB selector table.
template <int W, int ROWS> struct TileGeo {
  static constexpr uint32_t kRowBytes = ROWS == 16 ? ((W == 2) ? 40u : (W == 4) ? 80u : 128u) : ((W == 2) ? 24u : (W == 4) ? 48u : 80u);
  static constexpr uint32_t kPairsAt = (uint32_t)ROWS * kRowBytes;
  static_assert(kRowBytes % (W == 2 ? 8u : 16u) == 0u && kPairsAt % 16u == 0u, "stage_span stores whole spans, pairs are read four words at a time");
};
constexpr uint32_t kTableAt = 32u * 24u + 512u;          // the selector table: behind the larger of the two tiles of 2-bit rows
constexpr uint32_t kTileBytes = kTableAt + 2048u;
static_assert(TileGeo<8, 32>::kPairsAt + 512u <= kTileBytes && TileGeo<4, 32>::kPairsAt + 512u <= kTileBytes && TileGeo<8, 16>::kPairsAt + 512u <= kTileBytes, "");

// Loader side: a lane drops its fetched span `span` of row `row`, and the span's pair, into the tile.
template <int W, int G, int ROWS>
__device__ inline void stage_span(const SpanData<W, G>& d, uint8_t* tile, uint32_t row, uint32_t span) {
  uint32_t* pairs_lds = reinterpret_cast<uint32_t*>(tile + TileGeo<W, ROWS>::kPairsAt);
  uint8_t* dst = tile + row * TileGeo<W, ROWS>::kRowBytes + span * (4u * W);
  if constexpr (W == 2) {
    *reinterpret_cast<u32x2*>(dst) = (u32x2){d.cw[0], d.cw[1]};
    // the span's four decoded values instead of its (scale, zero): x_k = fp16(fma(k, scale, zero))
    const float s = half_bits_to_float(d.pair & 0xFFFFu);
    const float z = half_bits_to_float(d.pair >> 16);
    reinterpret_cast<u32x2*>(pairs_lds)[span * ROWS + row] = (u32x2){decode_pair(0.0f, 1.0f, s, z), decode_pair(2.0f, 3.0f, s, z)};
  } else {
#pragma unroll
    for (int h = 0; h < W / 4; ++h)
      reinterpret_cast<u32x4*>(dst)[h] = (u32x4){d.cw[4 * h], d.cw[4 * h + 1], d.cw[4 * h + 2], d.cw[4 * h + 3]};
    // as the decoder wants them: scale * 2^24 and zero
    reinterpret_cast<u32x2*>(pairs_lds)[span * ROWS + row] =
        (u32x2){__float_as_uint(half_bits_to_float(d.pair & 0xFFFFu) * 16777216.0f), __float_as_uint(half_bits_to_float(d.pair >> 16))};
  }
}

// Reader side, 16 rows: lane (a, kt) picks up the pieces "row 4 kt + i, columns 8 a .. 8 a + 7", i = 0 .. 3, and decodes them
// into t[i][m] = {X[4 kt + i][8 a + 2 m], X[4 kt + i][8 a + 2 m + 1]}.
template <int W>
__device__ inline void pieces_from_tile(const uint8_t* tile, const uint8_t* table, uint32_t a, uint32_t kt, uint32_t (&t)[4][4]) {
  constexpr uint32_t kRowBytes = TileGeo<W, 16>::kRowBytes;
  const uint32_t* pairs_lds = reinterpret_cast<const uint32_t*>(tile + TileGeo<W, 16>::kPairsAt);
  if constexpr (W == 2) {
    // by selection: the piece's two code bytes index the selector table, the selectors pick the values out of the row's four
    const u32x4* xs = reinterpret_cast<const u32x4*>(pairs_lds) + ((a >> 2) * 16u + 4u * kt) / 2u;
    const u32x4 x01 = xs[0], x23 = xs[1];  // the four-value tables of rows 4 kt .. 4 kt + 3 for this lane's columns
    const uint32_t xl[4] = {x01.x, x01.z, x23.x, x23.z}, xh[4] = {x01.y, x01.w, x23.y, x23.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t piece = *reinterpret_cast<const uint16_t*>(tile + (4u * kt + i) * kRowBytes + a * 2u);
      const u32x2 s0 = *reinterpret_cast<const u32x2*>(table + byte_times8<0>(piece));
      const u32x2 s1 = *reinterpret_cast<const u32x2*>(table + byte_times8<1>(piece));
      t[i][0] = __builtin_amdgcn_perm(xh[i], xl[i], s0.x);
      t[i][1] = __builtin_amdgcn_perm(xh[i], xl[i], s0.y);
      t[i][2] = __builtin_amdgcn_perm(xh[i], xl[i], s1.x);
      t[i][3] = __builtin_amdgcn_perm(xh[i], xl[i], s1.y);
    }
  } else {
    const u32x4* pr = reinterpret_cast<const u32x4*>(pairs_lds) + ((a >> 2) * 16u + 4u * kt) / 2u;
    const u32x4 pr01 = pr[0], pr23 = pr[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint8_t* src = tile + (4u * kt + i) * kRowBytes + a * W;
      const float s = __uint_as_float((i < 2 ? pr01 : pr23)[2 * (i & 1)]), z = __uint_as_float((i < 2 ? pr01 : pr23)[2 * (i & 1) + 1]);
      if constexpr (W == 4) {
        decode_word<4>(*reinterpret_cast<const uint32_t*>(src), s, z, t[i]);
      } else {
        const u32x2 w = *reinterpret_cast<const u32x2*>(src);
        decode_word<8>(w.x, s, z, t[i]);
        decode_word<8>(w.y, s, z, t[i] + 2);
      }
    }
  }
}

// The same with 32 rows of 64 columns: the pieces "row 16 u + 4 kt + i, columns 4 a .. 4 a + 3" as
// t[i][2 u + m] = {X[16 u + 4 kt + i][4 a + 2 m], X[16 u + 4 kt + i][4 a + 2 m + 1]}.
template <int W>
__device__ inline void pieces_from_tile64(const uint8_t* tile, const uint8_t* table, uint32_t a, uint32_t kt, uint32_t (&t)[4][4]) {
  constexpr uint32_t kRowBytes = TileGeo<W, 32>::kRowBytes;
  const uint32_t* pairs_lds = reinterpret_cast<const uint32_t*>(tile + TileGeo<W, 32>::kPairsAt);
  // 2 bits: all codes, then all look-ups, then the selections.  Left to itself the compiler now and then waits for every look-up by
  // itself (uniform 2-bit cards, several tasks a wave: 6 % of a call).
  uint32_t piece[8];
  u32x2 select[8];
  if constexpr (W == 2) {
#pragma unroll
    for (int i = 0; i < 8; ++i) piece[i] = tile[(16u * (i >> 2) + 4u * kt + (i & 3)) * kRowBytes + a];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) select[i] = *reinterpret_cast<const u32x2*>(table + 8u * piece[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t row = 16u * u + 4u * kt, at = (a >> 3) * 32u + row;
    if constexpr (W == 2) {
      const u32x4* xs = reinterpret_cast<const u32x4*>(pairs_lds) + at / 2u;
      const u32x4 x01 = xs[0], x23 = xs[1];
      const uint32_t xl[4] = {x01.x, x01.z, x23.x, x23.z}, xh[4] = {x01.y, x01.w, x23.y, x23.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t[i][2 * u] = __builtin_amdgcn_perm(xh[i], xl[i], select[4 * u + i].x);
        t[i][2 * u + 1] = __builtin_amdgcn_perm(xh[i], xl[i], select[4 * u + i].y);
      }
    } else {
      const u32x4* pr = reinterpret_cast<const u32x4*>(pairs_lds) + at / 2u;
      const u32x4 pr01 = pr[0], pr23 = pr[1];
      const float s[4] = {__uint_as_float(pr01.x), __uint_as_float(pr01.z), __uint_as_float(pr23.x), __uint_as_float(pr23.z)};
      const float z[4] = {__uint_as_float(pr01.y), __uint_as_float(pr01.w), __uint_as_float(pr23.y), __uint_as_float(pr23.w)};
#pragma unroll
      for (int i = 0; i < 4; i += (W == 4 ? 2 : 1)) {
        const uint8_t* src = tile + (row + i) * kRowBytes + a * (W / 2u);
        if constexpr (W == 4) {                          // two rows' codes side by side
          const uint32_t both = *reinterpret_cast<const uint16_t*>(src) | ((uint32_t)*reinterpret_cast<const uint16_t*>(src + kRowBytes) << 16);
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const uint32_t even = (both >> (8 * m)) & 0x000F000Fu, odd = (both >> (8 * m + 4)) & 0x000F000Fu;
            t[i][2 * u + m] = pack_halves(fma_low(even, s[i], z[i]), fma_low(odd, s[i], z[i]));
            t[i + 1][2 * u + m] = pack_halves(fma_high(even, s[i + 1], z[i + 1]), fma_high(odd, s[i + 1], z[i + 1]));
          }
        } else {
          decode_word<8>(*reinterpret_cast<const uint32_t*>(src), s[i], z[i], t[i] + 2 * u);
        }
      }
    }
  }
}

// Pairs of columns turned into pairs of rows: b[e] = {X[4kt][8a+e], X[4kt+1][8a+e], X[4kt+2][8a+e], X[4kt+3][8a+e]}.
__device__ inline void turn_pieces(const uint32_t (&t)[4][4], u32x2 (&b)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;      // high or low halves of two words
    b[e] = (u32x2){__builtin_amdgcn_perm(t[1][e >> 1], t[0][e >> 1], sel), __builtin_amdgcn_perm(t[3][e >> 1], t[2][e >> 1], sel)};
  }
}
template <int W>
__device__ inline void operands_from_tile(const uint8_t* tile, const uint8_t* table, uint32_t a, uint32_t kt, u32x2 (&b)[8]) {
  uint32_t t[4][4];
  pieces_from_tile<W>(tile, table, a, kt, t);
  turn_pieces(t, b);
}

// ---- cross-lane helpers ------------------------------------------------------------------------

// The lane's number, worked out where it is asked for: what depends on it is not kept in registers from further up.
__device__ inline uint32_t lane_anew() {
  uint32_t lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
  return lane;
}

// What lanes of the wave wrote to LDS before is what others read behind it: the hardware keeps one wave's LDS accesses in order,
// and this, which is no instruction, keeps the compiler to it.
__device__ inline void lds_handover() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int CTRL>
__device__ inline float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
// maximum / sum over the 16 lanes of a row, left in every lane of the row (row_ror: 8, 4, 2, 1)
__device__ inline float row_max16(float v) {
  v = fmaxf(v, dpp_move<0x128>(v));
  v = fmaxf(v, dpp_move<0x124>(v));
  v = fmaxf(v, dpp_move<0x122>(v));
  return fmaxf(v, dpp_move<0x121>(v));
}
__device__ inline float row_sum16(float v) {
  v += dpp_move<0x128>(v);
  v += dpp_move<0x124>(v);
  v += dpp_move<0x122>(v);
  return v + dpp_move<0x121>(v);
}

// Lane (n, kq) holds four partial sums a_r, one per head r, each to be added up over the four
// lanes (n, 0 .. 3); returns in lane (n, kq) the total of head kq.  v_permlane32_swap hands the
// lower half of the wave its partner's first operand and the upper half its partner's second
// one; v_permlane16_swap does the same between neighbouring rows of 16.
__device__ inline float sum_over_quarters(float a0, float a1, float a2, float a3) {
  const auto s02 = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a0), __builtin_bit_cast(uint32_t, a2), false, false);
  const uint32_t s02x = s02[0], s02y = s02[1];
  const float u0 = __builtin_bit_cast(float, s02x) + __builtin_bit_cast(float, s02y);      // heads 0 | 2
  const auto s13 = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a1), __builtin_bit_cast(uint32_t, a3), false, false);
  const uint32_t s13x = s13[0], s13y = s13[1];
  const float u1 = __builtin_bit_cast(float, s13x) + __builtin_bit_cast(float, s13y);      // heads 1 | 3
  const auto sr = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, u0), __builtin_bit_cast(uint32_t, u1), false, false);
  const uint32_t srx = sr[0], sry = sr[1];
  return __builtin_bit_cast(float, srx) + __builtin_bit_cast(float, sry);
}

// ---- score pass over key planes grouped per channel ---------------------------------------------
//
// Uniform cards with group size 32 whose key spans hold the 32 tokens of one token block for ONE
// channel (section layout [plane][token block][channel][32 codes]).  The contraction over the head
// dimension then runs over the card's rows, exactly as the value pass contracts over tokens, and the
// same tile does the regrouping: a round is 16 channels x 4 token blocks (a super-block of 128
// tokens); loader lane (n, kq) fetches channel 16 r + n of token block kq, reader lane (a, kt) gets
// "channels 16 r + 4 kt .. + 3, tokens 8 a .. 8 a + 7 of the super-block" as eight operands, and
// the other MFMA operand is q[head][16 r + 4 kt .. + 3], exact in fp16 (one MFMA per operand).
// After head_dim / 16 rounds the lane holds the scores of its eight tokens: summed over its own
// channels only when NARROW (sum_over_quarters adds the four kt and leaves head kt), complete
// otherwise (the 16 x 16 x 16 product adds the four kt itself; the lane holds heads 4 kt .. + 3).
template <int W, bool NARROW, int DS>
__device__ __forceinline__ void score_pass_kc(const AttendArgs& a, const CardGeom& g, int c, uint32_t pair, uint32_t j0, uint32_t cnt,
                                     uint32_t slots, uint32_t lane, float* lds, uint32_t pitch, uint32_t R4, uint8_t* tile,
                                     const uint8_t* table) {
  static_assert(W == 2 || W == 4 || W == 8, "per-channel key groups exist at 2, 4 and 8 bits");
  constexpr uint32_t D = 32u * DS;
  constexpr int kRounds = (int)D / 16;                      // rounds per super-block
  constexpr int kAhead = (W == 2) ? 4 : 2;                  // rounds whose loads are in flight; divides kRounds
  const uint32_t n = lane & 15u, kq = lane >> 4;
  const uint32_t R = a.rep;
  const uint32_t head = NARROW ? (n & 3u) : n;
  f16x4 qa[kRounds];
  {
    const uint32_t l = pair / g.kv_heads, hh = pair - l * g.kv_heads;
    const uint16_t* src = a.q + ((uint64_t)(l * a.q_heads + hh * R + (head < R ? head : 0u)) * D + 4u * kq);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      u32x2 raw = (u32x2)(0u);
      if (head < R) raw = *reinterpret_cast<const u32x2*>(src + 16 * r);
      qa[r] = __builtin_bit_cast(f16x4, raw);
    }
  }
  // first group (token block, channel 0) of the task's key plane: blocks of 32 tokens, head_dim groups each
  const uint64_t grp0 = ((uint64_t)pair * (g.tokens / 32u) + j0 / 32u) * D;
  const uint8_t* codes0 = a.card + g.off_codes[c];
  const uint8_t* pairs0 = a.card + g.off_meta[c];
  const auto fetch = [&](uint32_t sb, uint32_t r) {
    SpanData<W, 32> d;
#pragma unroll
    for (int i = 0; i < W; ++i) d.cw[i] = 0;
    d.pair = 0;
    const uint32_t tb = 4u * sb + kq;                        // token block inside the task
    if (32u * tb < cnt) {
      const uint64_t grp = grp0 + (uint64_t)tb * D + 16u * r + n;
      const uint8_t* src = codes0 + grp * (4u * W);
      if constexpr (W == 2) {
        const u32x2 t = *reinterpret_cast<const u32x2*>(src);
        d.cw[0] = t.x; d.cw[1] = t.y;
      } else {
#pragma unroll
        for (int h = 0; h < W / 4; ++h) {
          const u32x4 t = *reinterpret_cast<const u32x4*>(src + 16 * h);
          d.cw[4 * h] = t.x; d.cw[4 * h + 1] = t.y; d.cw[4 * h + 2] = t.z; d.cw[4 * h + 3] = t.w;
        }
      }
      d.pair = *reinterpret_cast<const uint32_t*>(pairs0 + grp * 4u);
    }
    return d;
  };
  SpanData<W, 32> buf[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) buf[u] = fetch(0u, (uint32_t)u);
  // every slot the softmax will read gets a value: `slots` is the task's token count rounded up to the softmax's
  // own granularity (at most the pitch), which can reach into a super-block that holds no token
  const uint32_t superblocks = (slots + 127u) / 128u;
  for (uint32_t sb = 0; sb < superblocks; ++sb) {
    f32x4 acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      stage_span<W, 32, 16>(buf[r % kAhead], tile, n, kq);
      buf[r % kAhead] = (r + kAhead < kRounds) ? fetch(sb, (uint32_t)(r + kAhead)) : fetch(sb + 1u, (uint32_t)(r + kAhead - kRounds));
      u32x2 b[8];
      operands_from_tile<W>(tile, table, n, kq, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const f16x4 be = __builtin_bit_cast(f16x4, b[e]);
        if constexpr (NARROW) acc[e] = __builtin_amdgcn_mfma_f32_4x4x4f16(qa[r], be, acc[e], 0, 0, 0);
        else acc[e] = __builtin_amdgcn_mfma_f32_16x16x16f16(qa[r], be, acc[e], 0, 0, 0);
      }
    }
    // tokens 128 sb + 8 a + e, e = 0 .. 7, of this lane
    const uint32_t t0 = 128u * sb + 8u * n;
    if constexpr (NARROW) {
      float sc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = sum_over_quarters(acc[e].x, acc[e].y, acc[e].z, acc[e].w);      // head kq
        sc[e] = (t0 + e < cnt) ? v * a.scale_log2 : -INFINITY;
      }
      float* dst = lds + kq * pitch + t0;
      if (t0 < pitch) *reinterpret_cast<f32x4*>(dst) = (f32x4){sc[0], sc[1], sc[2], sc[3]};
      if (t0 + 4u < pitch) *reinterpret_cast<f32x4*>(dst + 4) = (f32x4){sc[4], sc[5], sc[6], sc[7]};
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t r = 4u * kq + i;                      // the lane holds heads 4 kq .. 4 kq + 3
        if (r < R4) {
          float sc[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) sc[e] = (t0 + e < cnt) ? acc[e][i] * a.scale_log2 : -INFINITY;
          float* dst = lds + r * pitch + t0;
          if (t0 < pitch) *reinterpret_cast<f32x4*>(dst) = (f32x4){sc[0], sc[1], sc[2], sc[3]};
          if (t0 + 4u < pitch) *reinterpret_cast<f32x4*>(dst + 4) = (f32x4){sc[4], sc[5], sc[6], sc[7]};
        }
      }
    }
  }
}

// Raw value rows need no regrouping: the lane reads the pieces it needs - row 4 kt + i, dimensions 8 a .. 8 a + 7; with 64
// dimensions rows 4 kt + i and 16 + 4 kt + i, dimensions 4 a .. 4 a + 3 - where they lie.
template <int G, int DS>
__device__ inline SpanData<16, G> fetch_raw(const RowStream& s, uint32_t rd) {
  constexpr uint32_t kRow = RowBytes<16, DS>::kCodes;
  SpanData<16, G> d;
  d.pair = 0u;
  const uint32_t at = s.codes_at + rd * (RoundGeo<DS>::kTokens * kRow);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (DS == 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u32x2 t = buffer_load2(s.codes, at + (16u * h + i) * kRow);
        d.cw[8 * h + 2 * i] = t.x; d.cw[8 * h + 2 * i + 1] = t.y;
      }
    } else {
      const u32x4 t = buffer_load4(s.codes, at + i * kRow);
      d.cw[4 * i] = t.x; d.cw[4 * i + 1] = t.y; d.cw[4 * i + 2] = t.z; d.cw[4 * i + 3] = t.w;
    }
  }
  return d;
}

template <int W, int G, int DS>
__device__ inline RowStream value_stream(const uint8_t* card, const CardGeom& g, int c, uint64_t row0, uint32_t cnt, uint32_t n, uint32_t kq, uint32_t sl) {
  RowStream s = row_stream<W, G, DS>(card, g, c, row0, cnt, RoundGeo<DS>::row(n, kq), 4u * sl + RoundGeo<DS>::span(kq));
  if constexpr (W == 16) s.codes_at = 4u * kq * RowBytes<16, DS>::kCodes + (DS == 2 ? 8u * n : 256u * sl + 16u * n);
  return s;
}

template <int W, int G, int DS>
__device__ inline SpanData<W, G> fetch_value(const RowStream& s, uint32_t rd) {
  if constexpr (W == 16) return fetch_raw<G, DS>(s, rd);
  else return fetch_span<W, G, DS>(s, rd);
}

// Rounds whose loads are in flight ahead of the arithmetic: as many as the registers allow (a fetched span is 3 / 5 / 9 / 16
// registers at 2 / 4 / 8 / 16 bits; two slabs in flight cost twice that).  Their tokens, 64 at most, divide the units that tasks are
// made of, so that a padded round stays inside its task's LDS.
template <int W, int DS> struct Prefetch {
  static constexpr int kRounds = DS != 4 ? (W <= 4 ? 2 : 1) : W == 2 ? 4 : W == 4 ? 3 : W == 8 ? 2 : 1;
  static constexpr uint32_t kTokens = (uint32_t)kRounds * RoundGeo<DS>::kTokens;
};
template <int DS> constexpr bool whole_groups() {
  const uint32_t* unit = kUnit[DS / 4];
  return unit[0] % Prefetch<2, DS>::kTokens == 0u && unit[1] % Prefetch<4, DS>::kTokens == 0u && unit[2] % Prefetch<8, DS>::kTokens == 0u &&
         unit[3] % Prefetch<16, DS>::kTokens == 0u;
}
static_assert(whole_groups<2>() && whole_groups<4>() && whole_groups<8>(), "a task is a whole number of groups of rounds");

// How the value pass fills its MFMAs (see attend_task) and what it accumulates.
template <int HB, int DS> struct ValueGeo {
  static constexpr bool kTurned = HB == 2 && DS >= 4;
  static constexpr int kBlocks = HB == 2 && !kTurned ? 2 : 1;          // of 8 heads
  static constexpr int kSums = kTurned ? 8 : DS == 2 ? 2 : 4;          // pairs of dimensions, or dimensions
};

// fetch(0), fetch(1), ...: kept in this order and in one piece each.
template <int N, typename F>
__device__ __forceinline__ void first_fetches(const F& fetch) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    fetch(u);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// One sweep over a task's value rows: acc[b][m] += weights . V^, 2048 values a round.  `buf` holds the first rounds.
// The other parity's zero weights turn a value that is no number, or an infinity, into NaN in the dimension beside
// it: ISOLATE clears one half of every pair of dimensions (`keep`) to work the two out apart.
template <int W, int G, int HB, int DS, bool ISOLATE>
__device__ __forceinline__ void value_sweep(const RowStream& rows, SpanData<W, G> (&buf)[Prefetch<W, DS>::kRounds], uint32_t rounds, const float* lds,
                                   uint32_t pitch, uint32_t R4, uint8_t* tile, const uint8_t* table, uint32_t n, uint32_t kq, uint32_t keep,
                                   f32x4 (&acc)[ValueGeo<HB, DS>::kBlocks][ValueGeo<HB, DS>::kSums]) {
  constexpr int kPrefetch = Prefetch<W, DS>::kRounds;
  constexpr uint32_t kRows = RoundGeo<DS>::kTokens;
  constexpr bool kTurned = ValueGeo<HB, DS>::kTurned;
  constexpr int kBlocks = ValueGeo<HB, DS>::kBlocks, kSums = ValueGeo<HB, DS>::kSums, kHalves = DS == 2 ? 2 : 1;
  // a row of A has its parity's half of every word, and zero in the other: token 2 x sits in the low half of a pair of weights
  const uint32_t odd = n & 1u;
  const uint32_t sel[2] = {odd ? 0x01000C0Cu : 0x0C0C0100u, odd ? 0x03020C0Cu : 0x0C0C0302u};
  const uint32_t w_head = HB == 0 ? n >> 2 : kTurned ? n : n >> 1;     // of this lane's row (of the first block)
  const float* w_at = lds + w_head * pitch + 4u * kq + (HB == 0 ? (n & 2u) : 0u);
#pragma unroll
  for (int b = 0; b < kBlocks; ++b)
#pragma unroll
    for (int m = 0; m < kSums; ++m) acc[b][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (uint32_t rd0 = 0; rd0 < rounds; rd0 += kPrefetch) {
#pragma unroll
    for (int u = 0; u < kPrefetch; ++u) {                       // rounds past the task's end add zero weights times zeros
      const uint32_t rd = rd0 + u;
      __builtin_amdgcn_sched_barrier(0);                        // every round's loads stay in their round, see first_fetches
      uint32_t t[4][4];                                         // register i of operand x: row i of the lane's four
      if constexpr (W == 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int x = 0; x < 4; ++x) t[i][x] = DS == 2 ? buf[u].cw[8 * (x >> 1) + 2 * i + (x & 1)] : buf[u].cw[4 * i + x];
        buf[u] = fetch_raw<G, DS>(rows, rd + kPrefetch);
      } else {
        stage_span<W, G, (int)kRows>(buf[u], tile, RoundGeo<DS>::row(n, kq), RoundGeo<DS>::span(kq));
        buf[u] = fetch_span<W, G, DS>(rows, rd + kPrefetch);
        if constexpr (DS == 2) pieces_from_tile64<W>(tile, table, n, kq, t);
        else pieces_from_tile<W>(tile, table, n, kq, t);
      }
      if constexpr (kTurned) {
        u32x2 v[8];
        turn_pieces(t, v);
        u32x4 pw = (u32x4)(0u);
        if (w_head < R4) pw = *reinterpret_cast<const u32x4*>(w_at + rd * kRows);
        const f16x4 w_hi = __builtin_bit_cast(f16x4, (u32x2){pw.x, pw.y}), w_lo = __builtin_bit_cast(f16x4, (u32x2){pw.z, pw.w});
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const f16x4 ve = __builtin_bit_cast(f16x4, v[e]);
          acc[0][e] = __builtin_amdgcn_mfma_f32_16x16x16f16(w_hi, ve, acc[0][e], 0, 0, 0);
          acc[0][e] = __builtin_amdgcn_mfma_f32_16x16x16f16(w_lo, ve, acc[0][e], 0, 0, 0);
        }
        continue;
      }
      if constexpr (ISOLATE) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int x = 0; x < 4; ++x) t[i][x] &= keep;
      }
#pragma unroll
      for (int h = 0; h < kHalves; ++h) {
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
          const float* at = w_at + 8 * b * pitch + rd * kRows + 16 * h;
          u32x4 w_hi, w_lo;
          if constexpr (HB == 0) {                              // the lane's row is of high or of low parts
            const u32x2 pw = *reinterpret_cast<const u32x2*>(at);
#pragma unroll
            for (int i = 0; i < 4; ++i) w_hi[i] = __builtin_amdgcn_perm(0u, pw[i >> 1], sel[i & 1]);
          } else {
            u32x4 pw = (u32x4)(0u);
            if (b == 0 || 8u + w_head < R4) pw = *reinterpret_cast<const u32x4*>(at);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              w_hi[i] = __builtin_amdgcn_perm(0u, pw[i >> 1], sel[i & 1]);
              w_lo[i] = __builtin_amdgcn_perm(0u, pw[2 + (i >> 1)], sel[i & 1]);
            }
          }
#pragma unroll
          for (int m = 0; m < (DS == 2 ? 2 : 4); ++m) {
            const int x = DS == 2 ? 2 * h + m : m;
            const f16x8 v = __builtin_bit_cast(f16x8, (u32x4){t[0][x], t[1][x], t[2][x], t[3][x]});
            acc[b][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w_hi), v, acc[b][m], 0, 0, 0);
            if constexpr (HB > 0) acc[b][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w_lo), v, acc[b][m], 0, 0, 0);
          }
        }
      }
    }
  }
}

// Softmax over a task's tokens, four heads at a time: row kq of the wave takes head 4 hg + kq, its lane n the tokens
// 64 i + 4 n .. + 3 (the wave's own LDS accesses are in order).  Weights take the scores' places, `ml` the maximum and sum of every head.
// SCALED: the scale is applied here.
template <bool SCALED>
__device__ __forceinline__ void softmax_pass(float scale, uint32_t cnt, uint32_t slots, uint32_t n, uint32_t kq, float* lds, uint32_t pitch,
                                             uint32_t R4, float* ml) {
  const uint32_t whole = cnt & ~63u;                       // tokens of blocks that need no mask
  for (uint32_t hg = 0; hg < R4; hg += 4u) {
    const uint32_t r = hg + kq;
    float* row_w = lds + r * pitch;
    float m = -INFINITY;
    const auto top = [&](uint32_t t, bool masked) {
      const f32x4 sv = *reinterpret_cast<const f32x4*>(row_w + t);
#pragma unroll
      for (int i = 0; i < 4; ++i) m = fmaxf(m, !masked || t + i < cnt ? sv[i] : -INFINITY);
    };
    for (uint32_t t = 0; t < whole; t += 64u) top(t + 4u * n, false);
    for (uint32_t t = whole + 4u * n; t < slots; t += 64u) top(t, true);
    const float largest = row_max16(m);
    m = largest * scale;
    // Weights are 2^(score * scale - m).  With the difference to the largest score taken first, `rest` is what rounding m itself left over,
    // common to all of them, and a weight of 1 stays one of 2^rest.  As one rounding of score * scale - m that rest decided everything where
    // m is large: at 2^26 it is half an ulp, 4, and takes the weights out of fp16's range.  From 2^22 on, where it can be more than 1/4,
    // it is cut off: m is no nearer to the largest score than that anyway.  One subtraction a weight, 0.3 % of a call (short cards
    // of 16 heads 1 %); a second way for large m, behind a branch, cost the short calls 1 .. 2 %.
    const float rest = __builtin_amdgcn_fmed3f(__builtin_fmaf(largest, scale, -m), -0.25f, 0.25f);
    float l = 0.f;
    const auto weigh = [&](uint32_t t, bool masked) {
      const f32x4 sv = *reinterpret_cast<const f32x4*>(row_w + t);
      float ps[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = SCALED ? __builtin_fmaf(sv[i] - largest, scale, rest) : sv[i] - m;
        const float p = __builtin_amdgcn_exp2f(!masked || t + i < cnt ? x : -INFINITY);
        l += p;
        ps[i] = p * 16384.0f;
      }
      // what the value pass feeds the MFMA: p * 2^14 as an fp16 high part and the fp16 remainder (a normal number for any p
      // that matters), in the scores' places: four high parts, then four remainders
      const uint32_t h01 = pack_halves(ps[0], ps[1]), h23 = pack_halves(ps[2], ps[3]);
      *reinterpret_cast<u32x4*>(row_w + t) =
          (u32x4){h01, h23, pack_halves(fma_low(h01, -1.0f, ps[0]), fma_high(h01, -1.0f, ps[1])),
                  pack_halves(fma_low(h23, -1.0f, ps[2]), fma_high(h23, -1.0f, ps[3]))};
    };
    for (uint32_t t = 0; t < whole; t += 64u) weigh(t + 4u * n, false);
    for (uint32_t t = whole + 4u * n; t < slots; t += 64u) weigh(t, true);
    l = row_sum16(l);
    if (n == 0) *reinterpret_cast<float2*>(ml + 2u * r) = make_float2(m, l);
  }
}

// Scores of 64 dimensions once more, where a head's weights do not add up to a number: a zero of q times an infinity or a NaN in
// the key of the one token of a contraction is NaN in the other one's score.  Here each half of the contraction is
// multiplied with the other half of the keys cleared, so that zeros only meet zeros; scores that are numbers come out as before,
// to the bit.
template <int W, int G, int HB>
__device__ __forceinline__ void scores_apart(const RowStream& keys, __amdgpu_buffer_rsrc_t q_rows, uint32_t q_flip, uint32_t rounds, uint32_t n,
                                             uint32_t kq, float* lds, uint32_t pitch, uint32_t R4) {
  const uint32_t head = HB < 2 ? (n & 7u) : n;
#pragma unroll 1
  for (uint32_t half = 0; half < 2u; ++half) {              // tokens 0 .. 15 of every round, then tokens 16 .. 31
    const bool mine = (kq >> 1) == half;
    u32x4 q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = buffer_load4(q_rows, mine ? head * 128u + 64u * (kq & 1u) + 16u * j : 0x40000000u) ^ q_flip;
    if constexpr (W == 2) order_q2(q);
#pragma unroll 1
    for (uint32_t rd = 0; rd < rounds; ++rd) {
      uint32_t kb[16];
      if constexpr (W == 2) decode_fetched_bytes<G>(fetch_span<W, G, 2>(keys, rd), kb);
      else decode_fetched<W, G>(fetch_span<W, G, 2>(keys, rd), kb);
      f32x4 acc[2] = {(f32x4)(0.f), (f32x4)(0.f)};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x4 k4 = {kb[4 * j], kb[4 * j + 1], kb[4 * j + 2], kb[4 * j + 3]};
        acc[j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, mine ? k4 : (u32x4)(0u)), __builtin_bit_cast(f16x8, q[j]), acc[j & 1], 0, 0, 0);
      }
      if (head < R4 && (HB == 2 || n < 8u)) *reinterpret_cast<f32x4*>(lds + head * pitch + rd * 32u + 16u * half + 4u * kq) = acc[0] + acc[1];
    }
  }
}

// attend_kernel's arguments (one AttendArgs, so they lie where its argument segment begins), read where they are asked for: none of
// them is kept in registers from further up.
typedef const __attribute__((address_space(4))) AttendArgs* ArgsAnew;
__device__ inline ArgsAnew args_anew() {
  ArgsAnew at = (ArgsAnew)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(at));
  return at;
}

// Where a task's sums over values are no numbers: if a head's weights do not add up to one, its scores may be their neighbours' doing, and
// scores and softmax are worked out again.  Lane, arguments and the card's geometry are asked for anew, since what this rarely taken
// way keeps in registers is missed by the other (several tasks a wave, 64 dimensions: 3 % of a call).
template <int W, int G, int HB>
__device__ __forceinline__ void score_again(uint32_t pair, uint32_t j0, uint32_t cnt, uint32_t rounds, uint32_t slots, float* lds, float* ml) {
  constexpr int c = W == 2 ? 0 : W == 4 ? 1 : W == 8 ? 2 : 3;
  const uint32_t lane = lane_anew(), n = lane & 15u, kq = lane >> 4;
  const ArgsAnew a = args_anew();
  const uint32_t R = a->rep, R4 = HB == 0 ? 4u : ((R + 3u) & ~3u), pitch = a->chunk;
  const float l = ml[2u * min(n, R - 1u) + 1u];
  if (__builtin_amdgcn_ballot_w64(!(l == l)) == 0ull) return;
  const qkv_card_header_t* header = reinterpret_cast<const qkv_card_header_t*>(a->card);
  CardGeom g;                                              // what row_stream asks for
  if constexpr (W == 16) {
    g.off_fp16 = header->off_fp16;
  } else {
    g.off_codes[c] = header->off_codes[c];
    g.off_meta[c] = header->off_meta[c];
  }
  const RowStream keys = row_stream<W, G, 2>(a->card, g, c, (uint64_t)pair * header->count[c] + j0, cnt, RoundGeo<2>::row(n, kq), RoundGeo<2>::span(kq));
  const __amdgpu_buffer_rsrc_t q_rows = bounded(reinterpret_cast<const uint8_t*>(a->q + (uint64_t)pair * R * 64u), R * 128u);
  scores_apart<W, G, HB>(keys, q_rows, a->q_flip, rounds, n, kq, lds, pitch, R4);
  lds_handover();
  softmax_pass<true>(a->scale_log2, cnt, slots, n, kq, lds, pitch, R4, ml);
  lds_handover();
}

// One task: rows [j0, j1) of class c for the pair (layer, kv head) = pair.
// lds: scores / weights as [head][pitch] floats (R4 * pitch <= kLdsFloatsPerWave);
// tile: a round's packed rows followed by the rows' pairs.
//
// Both contractions run on v_mfma_f32_16x16x32_f16, 512 values of K^ or V^ an instruction.
//   scores   A = K^[token n][8 dimensions of the lane's span], B = q[head n][the same]: lane (n, kq) gets tokens 4 kq .. + 3 of
//            head n.  With 64 dimensions a round has 32 tokens; the two halves of the contraction belong to different
//            tokens, and q is zero in one of them: columns 0 .. 7 are the heads against tokens 0 .. 15, columns 8 .. 15 the
//            heads against tokens 16 .. 31 (more than 8 heads: one product for each half).  Zeros do not keep a key that is an
//            infinity or no number from the other token's score: see scores_apart.  Keys have a few dimensions
//            far larger than the others, and a sum that holds one of them rounds all that follows: two sums, added up
//            at the end, are nearer to the value in 64 bits (one sum: output 4.1 .. 6.8e-7 from it, two: 3.4 .. 4.9e-7).
//   values   V^ is decoded in pairs of neighbouring dimensions, and the contraction runs over (token, parity): B = {four
//            tokens x both dimensions of pair m}, and a row of A holds the weights of one head in the places of one
//            parity and zeros in the others.  So nothing has to be turned from pairs of dimensions into pairs of
//            tokens, and the rows of A that up to 4 heads leave free take that up: HB = 0 has rows (head, high or low part of
//            the weight, parity), HB = 1 (5 .. 8 heads) rows (head, parity) and an instruction each for the high and
//            the low parts, HB = 2 (9 .. 16 heads) two blocks of 8 heads with 64 dimensions; with more, where two blocks'
//            sums leave room for three waves a SIMD only (16 heads, 3622 tokens of 256 pairs: 75.3 -> 81.7 us), the
//            pairs are turned and v_mfma_f32_16x16x16_f16 has the 16 heads as rows.
// No accumulator sees both shapes: the compiler (ROCm 7.2) puts nothing between a 16 x 16 x 16 and a 16 x 16 x 32 product that start from each
// other's result, and one right behind the other, in either order, left 128 of 256 sums wrong in a program of just the two (with
// other products in between, none).
//
// DS = head_dim / 32 spans per token.  The lane mapping covers a slab of 128 dimensions (4 spans); head_dim 256 is two
// slabs (the score of a round adds both up before it is stored, the value pass sweeps the task once per slab).
// TURNS: a wave's later tasks add to the partial that the earlier ones left: its sums in part_o, where every lane finds its own, its
// maximum and sum of every head in LDS (`run`), since one lane writes them and sixteen read them.
template <int W, int G, int HB, int DS, bool KC, bool TURNS>
__device__ __forceinline__ void attend_task(const AttendArgs& a, const CardGeom& g, int c, uint32_t pair, uint32_t j0, uint32_t j1,
                                   uint32_t lane, float* lds, uint8_t* tile, uint8_t* table, float* ml, float* run, float* part_o, float* part_ml, bool first) {
  const uint32_t n = lane & 15u, kq = lane >> 4;          // also (a, kt) of the value pass
  const uint32_t R = a.rep, R4 = HB == 0 ? 4u : ((R + 3u) & ~3u);
  const uint32_t pitch = a.chunk;                          // of a head's scores in LDS
  const uint32_t lh = g.planes >> 1;
  const uint32_t n_c = g.n[c];
  const uint64_t k_row0 = (uint64_t)pair * n_c;            // K plane p = pair, V plane p = L*H + pair
  const uint64_t v_row0 = (uint64_t)(lh + pair) * n_c;
  const uint32_t cnt = j1 - j0;
  constexpr uint32_t kRows = RoundGeo<DS>::kTokens;
  const uint32_t rounds = (cnt + kRows - 1u) / kRows;
  constexpr int kPrefetch = Prefetch<W, DS>::kRounds;
  constexpr int S = (DS + 3) / 4;                          // slabs of 128 dimensions
  constexpr uint32_t D = 32u * DS;
  const uint32_t row = RoundGeo<DS>::row(n, kq), span = RoundGeo<DS>::span(kq);
  // Rounds are processed in whole groups of kPrefetch; a task is a whole number of such groups or ends with its class, so the
  // padded rounds stay inside the task's share of LDS.  The softmax covers `slots` tokens, those past the task's end at -inf.
  const uint32_t slots = (rounds + kPrefetch - 1) / kPrefetch * kPrefetch * kRows;
  if constexpr (KC) {
    if constexpr (W != 16 && G == 32 && DS <= 4)
      score_pass_kc<W, HB == 0, DS>(a, g, c, pair, j0, cnt, slots, lane, lds, pitch, R4, tile, table);
  } else {
    RowStream ks[S];
#pragma unroll
    for (int sl = 0; sl < S; ++sl) ks[sl] = row_stream<W, G, DS>(a.card, g, c, k_row0 + j0, cnt, row, 4u * sl + span);

    // ---- q as MFMA operands: operand j of slab sl is q[head][128 sl + 32 span + 8 j .. + 7].  Heads that do not exist, and the half of
    // a column that belongs to other tokens, lie past the end of the pair's rows of q and read as zero.
    constexpr int kSets = DS == 2 && HB == 2 ? 2 : 1;
    const uint32_t head = DS == 2 && HB < 2 ? (n & 7u) : n;
    const __amdgpu_buffer_rsrc_t q_rows = bounded(reinterpret_cast<const uint8_t*>(a.q + (uint64_t)pair * R * D), R * D * 2u);
    const uint32_t q_at = DS != 2 || HB == 2 || (n >> 3) == (kq >> 1) ? (head * D + 32u * span) * 2u : 0x40000000u;
    u32x4 raws[S][4];
#pragma unroll
    for (int sl = 0; sl < S; ++sl)
#pragma unroll
      for (int j = 0; j < 4; ++j) raws[sl][j] = buffer_load4(q_rows, q_at + 256u * sl + 16u * j);
    // The loads of the next kPrefetch rounds are always in flight.  They are issued in the order in which the loop issues them:
    // loads return in order, and what the loop's first round waits for is decided by the less favourable of the two orders.
    SpanData<W, G> buf[kPrefetch][S];
    first_fetches<kPrefetch>([&](int u) {
#pragma unroll
      for (int sl = 0; sl < S; ++sl) buf[u][sl] = fetch_span<W, G, DS>(ks[sl], u);
    });
    f16x8 qa[S * kSets][4];
#pragma unroll
    for (int sl = 0; sl < S; ++sl) {
      u32x4 (&raw)[4] = raws[sl];
#pragma unroll
      for (int j = 0; j < 4; ++j) raw[j] ^= a.q_flip;
      if constexpr (W == 2) order_q2(raw);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (kSets == 2) {
          qa[0][j] = __builtin_bit_cast(f16x8, kq < 2u ? raw[j] : (u32x4)(0u));
          qa[1][j] = __builtin_bit_cast(f16x8, kq < 2u ? (u32x4)(0u) : raw[j]);
        } else {
          qa[sl][j] = __builtin_bit_cast(f16x8, raw[j]);
        }
      }
    }

    // ---- scores: lds[head * pitch + token], not scaled yet
#pragma unroll 1
    for (uint32_t rd0 = 0; rd0 < rounds; rd0 += kPrefetch) {
#pragma unroll
      for (int u = 0; u < kPrefetch; ++u) {
        const uint32_t rd = rd0 + u;
        f32x4 acc[kSets][2];                             // a sum for every other operand, see below
#pragma unroll
        for (int s = 0; s < kSets; ++s)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[s][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < S; ++sl) {
          uint32_t kb[16];
          if constexpr (W == 2) decode_fetched_bytes<G>(buf[u][sl], kb);
          else decode_fetched<W, G>(buf[u][sl], kb);
          buf[u][sl] = fetch_span<W, G, DS>(ks[sl], rd + kPrefetch);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f16x8 kj = __builtin_bit_cast(f16x8, (u32x4){kb[4 * j], kb[4 * j + 1], kb[4 * j + 2], kb[4 * j + 3]});
#pragma unroll
            for (int s = 0; s < kSets; ++s) acc[s][j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kj, qa[kSets == 2 ? s : sl][j], acc[s][j & 1], 0, 0, 0);
          }
        }
        if (head < R4) {
          float* dst = lds + head * pitch + rd * kRows + 4u * kq;
#pragma unroll
          for (int s = 0; s < kSets; ++s)
            *reinterpret_cast<f32x4*>(dst + (kSets == 2 ? 16u * s : DS == 2 ? 16u * (n >> 3) : 0u)) = acc[s][0] + acc[s][1];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }   // per-token key groups

  // the first value rows are requested now, so that they arrive while the softmax runs
  RowStream vs = value_stream<W, G, DS>(a.card, g, c, v_row0 + j0, cnt, n, kq, 0u);
  SpanData<W, G> vbuf[kPrefetch];
  first_fetches<kPrefetch>([&](int u) { vbuf[u] = fetch_value<W, G, DS>(vs, u); });

  // the scores did without the selector table of 2-bit rows, and other widths' tiles lie over it
  if constexpr (W == 2 && !KC) build_select_table(reinterpret_cast<u32x2*>(table), lane);

  const float scale = KC ? 1.0f : a.scale_log2;            // not negative; scores of keys grouped per channel are scaled already
  lds_handover();                                          // scores
  softmax_pass<!KC>(scale, cnt, slots, n, kq, lds, pitch, R4, ml);
  lds_handover();                                          // weights, maxima and sums, the table

  // ---- values: one sweep over the task's rows per slab of 128 output dimensions (the weights stay in LDS)
  constexpr int kBlocks = ValueGeo<HB, DS>::kBlocks, kSums = ValueGeo<HB, DS>::kSums;
#pragma unroll 1
  for (int sl = 0; sl < S; ++sl) {
    if (sl > 0) {
      vs = value_stream<W, G, DS>(a.card, g, c, v_row0 + j0, cnt, n, kq, (uint32_t)sl);
      first_fetches<kPrefetch>([&](int u) { vbuf[u] = fetch_value<W, G, DS>(vs, u); });
    }
    f32x4 acc[kBlocks][kSums];
    value_sweep<W, G, HB, DS, false>(vs, vbuf, rounds, lds, pitch, R4, tile, table, n, kq, 0u, acc);
    if constexpr (!ValueGeo<HB, DS>::kTurned) {
      float finite = 0.f;                                    // stays 0 if all sums are numbers
#pragma unroll
      for (int b = 0; b < kBlocks; ++b)
#pragma unroll
        for (int m = 0; m < kSums; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) finite = __builtin_fmaf(acc[b][m][i], 0.0f, finite);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(finite != 0.0f) != 0ull, 0)) {
        if constexpr (DS == 2 && !KC) score_again<W, G, HB>(pair, j0, cnt, rounds, slots, lds, ml);
#pragma unroll 1
        for (uint32_t odd = 0; odd < 2u; ++odd) {
          f32x4 one[kBlocks][kSums];
#pragma unroll
          for (int u = 0; u < kPrefetch; ++u) vbuf[u] = fetch_value<W, G, DS>(vs, u);
          value_sweep<W, G, HB, DS, true>(vs, vbuf, rounds, lds, pitch, R4, tile, table, n, kq, odd ? 0xFFFF0000u : 0x0000FFFFu, one);
#pragma unroll
          for (int b = 0; b < kBlocks; ++b)
#pragma unroll
            for (int m = 0; m < kSums; ++m)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[b][m][i] = (uint32_t)(i & 1) == odd ? one[b][m][i] : acc[b][m][i];
        }
      }
    }
    // the lane holds: HB = 0 head kq, {high even, high odd, low even, low odd} of each pair of dimensions; turned: heads
    // 4 kq .. 4 kq + 3 of each dimension; otherwise heads 2 kq and 2 kq + 1 of every block, {even, odd} of both
    constexpr bool kTurned = ValueGeo<HB, DS>::kTurned;
    const uint32_t d0 = DS == 2 ? 4u * n : 128u * sl + 8u * n;
    constexpr float kUnscale = 1.0f / 16384.0f;
#pragma unroll
    for (int x = 0; x < (HB == 0 ? 1 : HB == 1 ? 2 : 4); ++x) {
      const uint32_t r = HB == 0 ? kq : kTurned ? 4u * kq + x : 8u * (x >> 1) + 2u * kq + (x & 1u);
      if (r < R) {
        float o[8];
#pragma unroll
        for (int e = 0; e < (DS == 2 ? 4 : 8); ++e) {
          const int m = e >> 1, h = e & 1;
          if constexpr (kTurned) o[e] = acc[0][e][x] * kUnscale;
          else if constexpr (HB == 0) o[e] = (acc[0][m][h] + acc[0][m][2 + h]) * kUnscale;
          else o[e] = acc[x >> 1][m][2 * (x & 1) + h] * kUnscale;
        }
        f32x4* dst = reinterpret_cast<f32x4*>(part_o + (r * D + d0));
        float2 now = *reinterpret_cast<const float2*>(ml + 2u * r);
        if (TURNS && !first) {                             // the wave's earlier tasks have left theirs here
          const float2 old = *reinterpret_cast<const float2*>(run + 2u * r);
          const f32x4 o0 = dst[0], o1 = DS != 2 ? dst[1] : (f32x4){0.f, 0.f, 0.f, 0.f};
          // a task whose weights do not add up to a positive number counts for nothing, here as in the merge
          const bool have = old.y > 0.f, add = now.y > 0.f;
          const float top = fmaxf(have ? old.x : -INFINITY, add ? now.x : -INFINITY);
          const float was = have ? __builtin_amdgcn_exp2f(old.x - top) : 0.f, is = add ? __builtin_amdgcn_exp2f(now.x - top) : 0.f;
          now = make_float2(top, (have ? old.y * was : 0.f) + (add ? now.y * is : 0.f));
#pragma unroll
          for (int e = 0; e < (DS == 2 ? 4 : 8); ++e) o[e] = __builtin_fmaf(have ? (e < 4 ? o0[e & 3] : o1[e & 3]) : 0.f, was, add ? o[e] * is : 0.f);
        }
        dst[0] = (f32x4){o[0], o[1], o[2], o[3]};
        if constexpr (DS != 2) dst[1] = (f32x4){o[4], o[5], o[6], o[7]};
        if (n == 0 && sl == S - 1) *reinterpret_cast<float2*>((TURNS ? run : part_ml) + 2u * r) = now;
      }
    }
  }
  if constexpr (TURNS) lds_handover();
}

// The lanes of a wave, for cut_tasks.
struct WaveLanes {
  __device__ inline uint32_t value(uint32_t v, uint32_t lane) const { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }
  __device__ inline uint32_t quad_sum(uint32_t v) const {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);        // quad_perm 1 0 3 2
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);  // quad_perm 2 3 0 1
  }
};

// KC: the card's key planes are grouped per channel (a uniform card at 2, 4 or 8 bits, group size 32).
// TURNS: there may be more tasks than waves.  An instance of its own, because what a loop around the tasks keeps in registers and
// takes apart again costs calls that have no use for it up to 1 us (16 pairs, 220 tokens, 5 heads 9.6 and 10.6 us; 4 pairs, 2570
// tokens of 256 dimensions 16.9 and 21.2).
template <int G, int HB, int DS, bool KC, bool TURNS>
__global__ __launch_bounds__(kWaveSize) __attribute__((amdgpu_waves_per_eu(4)))
void attend_kernel(AttendArgs a) {
  __shared__ __attribute__((aligned(16))) float lds[kLdsFloatsPerWave];
  // the value pass's LDS, 3.25 KiB: a round's packed rows (640 / 1280 / 2048 bytes at 2 / 4 / 8 bits; 64 dimensions 768 / 1536 / 2560),
  // then the rows' pairs (512 bytes), then at 2 bits the 2 KiB selector table
  __shared__ __attribute__((aligned(16))) uint8_t tiles[kTileBytes];
  __shared__ __attribute__((aligned(16))) float mls[32];      // the task's maximum and sum of every head
  __shared__ __attribute__((aligned(16))) float runs[TURNS ? 32 : 2];      // and the wave's, over its tasks so far
  CardGeom g;
  bool ok = card_geometry_from_header(a.card, a.card_bytes, a.layers, a.kv_heads, a.head_dim, a.group_size,
                                      a.tokens, g, KC ? QKV_FLAG_KEYS_PER_CHANNEL : 0u);
  if (KC && ok) {                              // the shapes the per-channel score pass is written for
    const bool uniform = g.n[0] == g.tokens || g.n[1] == g.tokens || g.n[2] == g.tokens;
    ok = uniform && g.group_size == 32u && g.head_dim <= 128u && g.tokens % (g.head_dim == 64u ? 64u : 32u) == 0u;
  }
  // the header's verdict, for the merging kernel that follows on the stream and for the caller
  const bool one = blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0;
  if (one) {
    if (!ok) *a.valid = 0u;
    if (a.status) *a.status = ok ? 0u : QKV_STATUS_BAD_HEADER;
  }
  if (!ok) return;                            // uniform over the grid
  const uint32_t gw = blockIdx.x;
  const uint32_t pairs = g.planes >> 1;
  // all pairs' first waves, then all second ones: a grid of pairs x waves where its height allows
  const uint32_t tau = a.flat ? gw / pairs : blockIdx.y, pair = a.flat ? gw - tau * pairs : gw;
  float* my_lds = lds;
  uint8_t* my_tile = tiles;
  uint8_t* my_table = my_tile + kTableAt;
  float* my_ml = mls;
  const TaskCut cut = cut_tasks<DS, KC>(a, g, threadIdx.x & 63u, WaveLanes());
  const uint32_t tasks = cut.tasks[0] + cut.tasks[1] + cut.tasks[2] + cut.tasks[3];
  if (one) *a.valid = min(tasks, a.waves);
  if (tau >= min(tasks, a.waves)) return;      // a spare wave: the merge knows
  const uint64_t part = (uint64_t)pair * a.waves + tau;
  float* part_o = reinterpret_cast<float*>(uniform64(reinterpret_cast<uint64_t>(a.part_o + part * a.rep * (32u * DS))));
  float* part_ml = reinterpret_cast<float*>(uniform64(reinterpret_cast<uint64_t>(a.part_ml + part * a.rep * 2u)));
#pragma unroll 1
  for (uint32_t t = tau; t < tasks; t += a.waves) {
    // the lane's number, worked out anew each time: it and what depends on it alone (q in two orders, offsets at four widths) would
    // otherwise be kept in registers that the loop does not have
    const uint32_t ln = TURNS ? lane_anew() : threadIdx.x;
    uint32_t j0 = 0, j1 = 0;
    const int cls = cut.find(g, t, j0, j1);
    const bool first = !TURNS || t == tau;
    if (cls == 0) {
      if (KC) build_select_table(reinterpret_cast<u32x2*>(my_table), ln);
      attend_task<2, G, HB, DS, KC, TURNS>(a, g, 0, pair, j0, j1, ln, my_lds, my_tile, my_table, my_ml, runs, part_o, part_ml, first);
    }
    if (cls == 1) attend_task<4, G, HB, DS, KC, TURNS>(a, g, 1, pair, j0, j1, ln, my_lds, my_tile, my_table, my_ml, runs, part_o, part_ml, first);
    if (cls == 2) attend_task<8, G, HB, DS, KC, TURNS>(a, g, 2, pair, j0, j1, ln, my_lds, my_tile, my_table, my_ml, runs, part_o, part_ml, first);
    if constexpr (!KC) {                       // a card grouped per channel has no raw rows
      if (cls == 3) attend_task<16, G, HB, DS, false, TURNS>(a, g, 3, pair, j0, j1, ln, my_lds, my_tile, my_table, my_ml, runs, part_o, part_ml, first);
    }
    if (!TURNS) break;                         // no more tasks than waves (see cut_parameters)
  }
  if constexpr (TURNS) {
    if (threadIdx.x < a.rep) reinterpret_cast<float2*>(part_ml)[threadIdx.x] = reinterpret_cast<const float2*>(runs)[threadIdx.x];
  }
}

// Merges the partials of one (layer, query head).  The tasks' weights relative to the common maximum are worked out once,
// a thread per task; then every group of head_dim / 4 threads adds up its share of the tasks, four output
// dimensions per thread, and the groups' sums are added in order.  Bound by the latency of one trip to the partials:
// one thread per dimension walking over all tasks, with the weights' exponentials in the loop, took 7.6 us at 8K tokens
// (25 tasks); this takes 5.8.  The number of partials and the weights of the first ones are asked for at the same time, and the
// grid is pairs x query heads, so that no division stands in front: a trip and two chains of thirty instructions less, whole
// call 1024 tokens of 256 pairs 18.7 -> 17.7 us, 300 tokens 14.25 -> 11.65, 1000 tokens of 32 pairs 11.9 -> 10.9.
// How many threads: merge_threads.
template <int kMergeThreads>
__global__ __launch_bounds__(kMergeThreads) void attend_merge_kernel(AttendArgs a) {
  constexpr int kMergeBatch = kMergeThreads;           // tasks whose weights are held in LDS at a time
  __shared__ float weight[kMergeBatch];
  __shared__ float part_max[kMergeThreads / kWaveSize], part_den[kMergeThreads / kWaveSize];
  __shared__ f32x4 sums[kMergeThreads];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, D = a.head_dim;
  const uint32_t pair = blockIdx.x, r = blockIdx.y;    // (layer, kv head) and query head of it
  const uint64_t lq = (uint64_t)pair * a.rep + r;      // (layer, query head)
  const uint64_t part0 = (uint64_t)pair * a.waves;
  // asked for together with the number of partials: those past it hold anything and are not looked at
  float2 ml = make_float2(-INFINITY, 0.f);
  if (tid < a.waves) ml = *reinterpret_cast<const float2*>(a.part_ml + ((part0 + tid) * a.rep + r) * 2);
  const uint32_t tasks = *a.valid;
  if (tasks == 0) return;                              // header refused: outputs stay untouched
  const uint32_t per = D / 4u, split = kMergeThreads / per;      // threads per task's row, tasks at a time
  const uint32_t mine = tid / per, d4 = tid - mine * per;
  float M = -INFINITY, den = 0.f;                      // running maximum, and sums relative to it
  f32x4 num = {0.f, 0.f, 0.f, 0.f};
  for (uint32_t t0 = 0; t0 < tasks; t0 += kMergeBatch) {
    const uint32_t nb = min((uint32_t)kMergeBatch, tasks - t0);
    float m = -INFINITY, lt = 0.f;
    if (tid < nb) {
      if (t0 != 0u) ml = *reinterpret_cast<const float2*>(a.part_ml + ((part0 + t0 + tid) * a.rep + r) * 2);
      if (ml.y > 0.f) { m = ml.x; lt = ml.y; }         // a partial whose weights do not add up to a positive number counts for nothing
    }
    float top = row_max16(m);
    top = fmaxf(top, __shfl_xor(top, 16, kWaveSize));
    top = fmaxf(top, __shfl_xor(top, 32, kWaveSize));
    if (lane == 0) part_max[wave] = top;
    __syncthreads();
    float Mb = M;
#pragma unroll
    for (int w = 0; w < kMergeThreads / kWaveSize; ++w) Mb = fmaxf(Mb, part_max[w]);
    const float rescale = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mb);
    M = Mb;
    const float w = lt > 0.f ? __builtin_amdgcn_exp2f(m - M) : 0.f;
    weight[tid] = lt > 0.f ? w : -1.f;                 // its sums are anything: not to be touched
    float wl = row_sum16(w * lt);
    wl += __shfl_xor(wl, 16, kWaveSize);
    wl += __shfl_xor(wl, 32, kWaveSize);
    if (lane == 0) part_den[wave] = wl;
    __syncthreads();
    den *= rescale;
#pragma unroll
    for (int x = 0; x < kMergeThreads / kWaveSize; ++x) den += part_den[x];
    num *= rescale;
#pragma unroll 4
    for (uint32_t t = mine; t < nb; t += split) {
      const float wt = weight[t];
      if (!(wt < 0.f)) num += wt * *reinterpret_cast<const f32x4*>(a.part_o + ((part0 + t0 + t) * a.rep + r) * D + 4u * d4);
    }
    if (t0 + kMergeBatch < tasks) __syncthreads();        // the weights are written again
  }
  sums[tid] = num;
  __syncthreads();
  if (tid < per) {
    for (uint32_t x = 1; x < split; ++x) num += sums[x * per + tid];
    *reinterpret_cast<f32x4*>(a.out + lq * D + 4u * tid) = num / den;
  }
  if (tid == 0 && a.lse) a.lse[lq] = (M + __builtin_log2f(den)) * 0.69314718055994530942f;
}

}  // namespace

// ---- scratch for callers that cannot allocate -------------------------------------------------
//
// qkv_card_attend_static keeps the partials in this array instead of a caller's workspace.  Every
// GPU the library runs on holds its own copy, at its own address, until the process ends.  In host
// code the array's name is only a handle for the runtime: the device address comes from
// hipGetSymbolAddress, once per device, and that address is what kernels and copies are given.
namespace {
constexpr uint64_t kStaticScratchBytes = QKV_ATTEND_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) float scratch[kStaticScratchBytes / sizeof(float)];
std::atomic<float*> g_scratch_at[64];        // per device ordinal, null = not looked up yet
}  // namespace

// The current device's copy of the scratch array.  Looks the address up on the first call per device.
hipError_t attend_static_scratch(float** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  float* p = g_scratch_at[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    void* at = nullptr;
    e = hipGetSymbolAddress(&at, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (at == nullptr) return hipErrorInvalidSymbol;
    p = static_cast<float*>(at);
    g_scratch_at[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return hipSuccess;
}

// Threads of a merging workgroup.  Few workgroups, or many partials each: 256, many partials are under way at once.  Else, with
// more workgroups than 256 threads each find room for: fewer, and one wave, which waits for no other, where that reads the
// partials in a few trips.  Merge alone, us, with 256 / 128 / 64 threads: head_dim 128, 1024 workgroups, 25 tasks 5.8 / 6.2 /
// 8.6; 1280, 17 tasks 5.9 / 5.4 / 6.5, 33 tasks 6.5 / 7.0 / 9.8; 1792, 400 tasks 75 / 97 / 146; 3072, 9 tasks 6.8 / 5.5 / 5.5, 65
// tasks 20.2 / 18.4 / 20.4, 129 tasks 41 / 48 / 61; 6144, 5 tasks 10.5 / 7.4 / 5.4; head_dim 64, 4096 workgroups, 9 tasks 8.8 / 5.9
// / 4.9, 65 tasks 14.5 / 14.5 / 15.6, 400 tasks 107 / 103 / 110; head_dim 256, 4096, 33 tasks 22.0 / 20.9 / 21.6, 129 140 / 145 / 150.
static uint32_t merge_threads(uint32_t workgroups, uint32_t tasks, uint32_t head_dim) {
  if (workgroups <= 1024u || tasks * head_dim > (workgroups <= 2048u ? 4096u : 9216u)) return 256u;
  return workgroups <= 2048u || tasks * head_dim / 4u > 256u ? 128u : 64u;
}

hipError_t launch_attend(const uint8_t* card, uint64_t card_bytes, const CardGeom& expect, const void* q,
                         uint32_t q_heads, float softmax_scale, float* out, float* lse, float* workspace,
                         uint64_t workspace_bytes, uint32_t* status, bool keys_per_channel, hipStream_t stream) {
  AttendArgs a;
  a.card = card;
  a.card_bytes = card_bytes;
  a.layers = expect.layers; a.kv_heads = expect.kv_heads; a.head_dim = expect.head_dim; a.group_size = expect.group_size;
  a.tokens = expect.tokens;
  a.q = static_cast<const uint16_t*>(q);
  a.q_heads = q_heads;
  a.rep = q_heads / expect.kv_heads;
  a.scale_log2 = softmax_scale * 1.44269504088896340736f;
  a.q_flip = !keys_per_channel && std::signbit(a.scale_log2) ? 0x80008000u : 0u;
  if (a.q_flip != 0u) a.scale_log2 = -a.scale_log2;
  const uint64_t pairs = (uint64_t)expect.layers * expect.kv_heads;
  const uint32_t D = expect.head_dim;
  const uint32_t partials = cut_parameters(a, expect.tokens, a.rep, pairs, D, keys_per_channel, workspace_bytes / sizeof(float));
  a.part_o = workspace;
  a.part_ml = workspace + pairs * a.waves * a.rep * D;
  a.valid = reinterpret_cast<uint32_t*>(workspace + pairs * a.waves * a.rep * (D + 2u));
  a.out = out;
  a.lse = lse;
  a.status = status;
  a.flat = a.waves > 65535u ? 1u : 0u;
  const dim3 grid(a.flat ? (uint32_t)(pairs * a.waves) : (uint32_t)pairs, a.flat ? 1u : a.waves), block(kWaveSize);
  const int hb = a.rep <= 4u ? 0 : a.rep <= 8u ? 1 : 2;      // how the weights fill the rows of an MFMA, see attend_task
  const uint32_t G = expect.group_size;
#define QKV_LAUNCH_ATTEND_T(GG, DSS, KCC, TT)                                                                      \
  do {                                                                                                             \
    if (hb == 0) hipLaunchKernelGGL((attend_kernel<GG, 0, DSS, KCC, TT>), grid, block, 0, stream, a);              \
    else if (hb == 1) hipLaunchKernelGGL((attend_kernel<GG, 1, DSS, KCC, TT>), grid, block, 0, stream, a);         \
    else hipLaunchKernelGGL((attend_kernel<GG, 2, DSS, KCC, TT>), grid, block, 0, stream, a);                      \
  } while (0)
#define QKV_LAUNCH_ATTEND(GG, DSS)                                                                                 \
  do {                                                                                                             \
    if (a.waves < partials) QKV_LAUNCH_ATTEND_T(GG, DSS, false, true); else QKV_LAUNCH_ATTEND_T(GG, DSS, false, false); \
  } while (0)
  if (keys_per_channel) {                      // the host has checked: group size 32, head_dim 64 or 128
    if (D == 64u) QKV_LAUNCH_ATTEND_T(32, 2, true, false); else QKV_LAUNCH_ATTEND_T(32, 4, true, false);
  } else if (D == 64u) {
    if (G == 32u) QKV_LAUNCH_ATTEND(32, 2); else QKV_LAUNCH_ATTEND(64, 2);
  } else if (D == 128u) {
    if (G == 32u) QKV_LAUNCH_ATTEND(32, 4); else if (G == 64u) QKV_LAUNCH_ATTEND(64, 4); else QKV_LAUNCH_ATTEND(128, 4);
  } else {
    if (G == 32u) QKV_LAUNCH_ATTEND(32, 8); else if (G == 64u) QKV_LAUNCH_ATTEND(64, 8); else QKV_LAUNCH_ATTEND(128, 8);
  }
#undef QKV_LAUNCH_ATTEND_T
#undef QKV_LAUNCH_ATTEND
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 merge_grid((uint32_t)pairs, a.rep);
  const uint32_t threads = merge_threads(expect.layers * q_heads, a.waves, D);
  if (threads == 64u) hipLaunchKernelGGL(attend_merge_kernel<64>, merge_grid, dim3(64), 0, stream, a);
  else if (threads == 128u) hipLaunchKernelGGL(attend_merge_kernel<128>, merge_grid, dim3(128), 0, stream, a);
  else hipLaunchKernelGGL(attend_merge_kernel<256>, merge_grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace qkv
