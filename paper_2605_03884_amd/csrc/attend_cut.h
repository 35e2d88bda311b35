// attend_cut.h — how attention over a card is cut into tasks and dealt to waves: what the host decides from the shape (the workspace's
// partials, the waves of a pair), and what the device decides from the card's class counts.  Plain C++ but for `QKV_CUT_FN`, so that
// a host program can go through it for any shape.  Internal to the GPU library.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "../../include/qkvcard.h"

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define QKV_CUT_FN __device__ inline
#else
#define QKV_CUT_FN inline
#endif

namespace qkv {

// Tokens of a group of rounds whose loads are in flight together (Prefetch), by class, at 64, 128 and 256 dimensions (there a
// multiple of them): what makes tasks of different widths last about as long.
constexpr uint32_t kUnit[3][4] = {{64u, 64u, 32u, 32u}, {64u, 48u, 32u, 16u}, {64u, 32u, 32u, 16u}};
constexpr uint32_t kLdsFloatsPerWave = 1536;             // scores of one task: chunk tokens x padded query heads (6 KiB)

constexpr uint64_t kWaveSlots = 256u * 4u * 4u;          // four waves on each of the four SIMDs of 256 compute units

// The least number of partials of a (layer, kv head) that a workspace has room for, and the rows of a task (`chunk`) that it goes by: as many
// as the scores of a task (tokens x query heads padded to a multiple of 4) may be in the wave's 6 KiB of LDS, in
// multiples of 192 that every unit of kUnit divides, or 64 where fewer than 192 fit.  The larger size means fewer partials and less
// work per task (90 us against 96 us at 8K tokens x 256 pairs); the smaller one is taken when the larger would
// not even fill the chip's wave slots once (four waves per SIMD, 256 compute units).  How many rows a task really gets: cut_tasks.
inline void attend_plan(uint64_t tokens, uint32_t rep, uint64_t pairs, uint32_t* chunk, uint32_t* max_tasks) {
  const uint32_t r4 = (rep + 3u) & ~3u;
  const uint32_t room = kLdsFloatsPerWave / r4;                 // tokens whose scores fit, 96 at least
  const uint32_t limit = room >= 192u ? room / 192u * 192u : 64u;
  uint32_t c = limit;
  while (c > 192u && pairs * ((tokens + c - 1) / c + 2u) < kWaveSlots) c -= 192u;
  *chunk = c;
  *max_tasks = (uint32_t)((tokens + *chunk - 1) / *chunk) + 3u;   // every class may end with a partly filled task
}

// The number of tasks that short sequences are better cut into, where the workspace has room for their partials: one
// per wave slot of the chip, but no more than there are units of work at a middling mix of widths (an empty task still
// costs its dispatch).  Only up to 4 query heads per kv head and head_dim 128: beyond, a task's fixed part and the merge are
// heavier, and the rule would need a line of its own.  Attention and merge, us, with the least number of tasks and cut like
// this (a pair's waves one after the other): 256 pairs, 8 heads, 300 tokens 20.2 and 18.8, 1000 29.6 and 25.0,
// 4000 55.2 and 55.4; 16 heads, 2000 tokens 51.5 and 53.8; 32 pairs, 8 heads, 1000 tokens 18.6 and 15.3, 4000 20.9 and 23.8;
// head_dim 256, 4 heads, 1000 23.7 and 19.2, 4000 29.9 and 35.5.
// And no more than 96: with few pairs the merge, a few workgroups that go through all partials, takes longer than what shorter
// tasks save.  Whole call, 4 heads and a mean over widths, us, with at most 1368 / 192 / 96 / 64: 1 pair, 8192 tokens 16 / 16 / 15 / 15,
// 32768 40 / 22 / 23 / 22, 65536 73 / 32 / 33 / 32; 8 pairs, 8192 19 / 19 / 17 / 17, 24000 39 / 26 / 23 / 23; 16 pairs, 12000 24 / 22 / 20 / 19.
// Not beyond the fixed scratch array, so that the call that uses it cuts its tasks - and rounds its sums - like the
// one with a workspace.
inline uint32_t attend_more_tasks(uint64_t tokens, uint32_t rep, uint64_t pairs, uint32_t head_dim, uint32_t max_tasks) {
  if (rep > 4u || head_dim > 128u) return max_tasks;
  uint64_t want = kWaveSlots / pairs;
  const uint64_t useful = tokens / 48u + 3u;
  if (want > useful) want = useful;
  if (want > 96u) want = 96u;
  const uint64_t fits = (QKV_ATTEND_STATIC_SCRATCH_BYTES / sizeof(float) - 4u) / (pairs * rep * (head_dim + 2u));
  if (want > fits) want = fits;
  return want > max_tasks ? (uint32_t)want : max_tasks;
}

// Waves per pair: all pairs' first waves are dealt out first, then all second ones: the holes that waves without a task leave are
// then one piece at the end (a pair's waves one after the other: 2000 tokens of 256 pairs 41.4 us, like this 26.8).  As many turns of the chip's wave slots as leave no more than a tenth of the last one empty, one if that
// does, but no more than `most`, the partials a pair has room for.
inline uint32_t waves_per_pair(uint64_t pairs, uint32_t most) {
  uint64_t w = 0;
  for (uint64_t turns = 1; turns <= 8u; ++turns) {
    w = turns * kWaveSlots / pairs;
    if (w >= most || 10u * w * pairs >= 9u * turns * kWaveSlots) break;
  }
  return (uint32_t)std::min<uint64_t>(most, w == 0u ? 1u : w);
}

// What a launch decides: the fields below of `a`, and the number of partials that its workspace (in floats) has room for, of a pair.
// Waves take several tasks each only where they are fewer than the partials; where they are as many, cut_tasks makes no more tasks than that
// (see there), and a wave takes one.
template <typename A>
inline uint32_t cut_parameters(A& a, uint64_t tokens, uint32_t rep, uint64_t pairs, uint32_t head_dim, bool keys_per_channel, uint64_t workspace_floats) {
  uint32_t partials = 0;
  attend_plan(tokens, rep, pairs, &a.rows, &partials);
  const uint32_t more = attend_more_tasks(tokens, rep, pairs, head_dim, partials);
  if (workspace_floats >= pairs * more * rep * (head_dim + 2u) + 4u) partials = more;
  // with keys grouped per channel every task has a wave of its own: there is no register left for more
  a.waves = keys_per_channel ? partials : waves_per_pair(pairs, partials);
  a.chunk = kLdsFloatsPerWave / ((rep + 3u) & ~3u) / 16u * 16u;
  // a group of rounds whose loads are in flight together; keys grouped per channel are scored 128 tokens at a time, in whole
  // blocks of 32: as many groups as are whole blocks, 128 tokens where LDS holds a multiple
  for (int c = 0; c < 4; ++c) a.unit[c] = kUnit[head_dim / 128u][c];
  if (keys_per_channel) {
    a.unit[0] = a.unit[1] = a.unit[2] = a.rows % 128u == 0u || (a.chunk >= 128u && tokens <= 128u * (uint64_t)partials) ? 128u : 64u;
    if (head_dim == 128u) a.unit[1] = 96u;
  }
  for (int c = 0; c < 4; ++c) {
    a.fit[c] = a.chunk / a.unit[c];
    a.fit_rows[c] = std::max(1u, a.rows / a.unit[c]);
  }
  return partials;
}

QKV_CUT_FN uint32_t lower(uint32_t a, uint32_t b) { return a < b ? a : b; }
QKV_CUT_FN uint32_t higher(uint32_t a, uint32_t b) { return a > b ? a : b; }

// How a card's rows are cut into the tasks of a (layer, kv head).
//
// Where it can be, all tasks get the same number of units: a unit is one group of rounds whose loads are in flight
// together - fewer tokens at larger widths - so a task lasts about as long whatever its width.  s units a task make at
// most k - 1 + (sum u_c - (k - 1)) / s tasks (rounded up) of the k classes present, so s >= (sum u_c - (k - 1)) / (n - (k - 1)) keeps
// them within n.  In this order, with n the waves of a pair:
//   one turn of even tasks; then with no more than `rows` rows each, the length that the workspace's partials go by (a chip that
//   is not full is bound by latency, and a wide row takes little longer than a narrow one); then as many rows as that of any width;
//   up to three turns of even tasks, where LDS holds three units or more: the waves run in step, and one that got two long tasks
//   while others have one holds up the call;
//   beyond, the longest tasks that LDS holds: a task's start and end cost about 3 us that four waves a SIMD do not quite hide (32K
//   tokens of 2 bits with tasks of 192 rows 218 us, of 384 199).
// Where the waves are as many as the partials, one of the first three, or the last, makes no more tasks than that: units divide `rows`, or,
// where `rows` is 64 and holds one unit of 48 (4 bits, 128 dimensions, 9 .. 16 heads), tasks of LDS's 96 rows or more are fewer.
// Whole call, us, with one task a wave, more of them than wave slots, and like this: 8192 tokens at budget 3 of 256 pairs 72 and 65, 224
// pairs 65 and 59, 9000 tokens 77 and 71, 5000 tokens 48.6 and 40; 512 pairs, 9000 tokens 140 and 137.
struct TaskCut {
  uint32_t tasks[4];       // of each class
  uint32_t step[4];        // rows of a task
  // Class of task `tau` and its rows [j0, j1); -1: there is no such task.
  template <typename G>
  QKV_CUT_FN int find(const G& g, uint32_t tau, uint32_t& j0, uint32_t& j1) const {
    int cls = -1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (cls < 0) {
        if (tau < tasks[c]) {
          cls = c;
          j0 = tau * step[c];
          j1 = lower(g.n[c], j0 + step[c]);
        } else {
          tau -= tasks[c];
        }
      }
    }
    return cls;
  }
};

QKV_CUT_FN uint32_t divide_up(uint32_t a, uint32_t b) { return (a + b - 1u) / b; }

// Every wave goes through this between the header and its first load, and a division is a chain of some thirty dependent
// instructions: lane 4 k + c works on class c of candidate k, so that all that can be divided at the same time is.
// `wave` gives what other lanes hold: value(v, lane), and quad_sum(v) over four neighbouring lanes.
template <int DS, bool KC, typename A, typename G, typename W>
QKV_CUT_FN __attribute__((always_inline)) TaskCut cut_tasks(const A& a, const G& g, uint32_t lane, W&& wave) {
  uint32_t units[4], sum = 0, present = 0, most = ~0u, room = ~0u;      // units of every class present that fit `rows`, and LDS
  const uint32_t c = lane & 3u, k = lane >> 2;
  uint32_t my_unit = 0, my_units = 0, my_fit = 0, my_fit_rows = 0;
#pragma unroll
  for (uint32_t x = 0; x < 4u; ++x) {
    const uint32_t unit = KC ? a.unit[x] : kUnit[DS / 4][x];
    units[x] = KC ? (g.n[x] == 0u ? 0u : divide_up(g.n[x], unit)) : divide_up(g.n[x], unit);
    sum += units[x];
    present += (uint32_t)(g.n[x] != 0u);
    most = g.n[x] == 0u ? most : lower(most, a.fit_rows[x]);
    room = g.n[x] == 0u ? room : lower(room, a.fit[x]);
    my_unit = c == x ? unit : my_unit;
    my_units = c == x ? units[x] : my_units;
    my_fit = c == x ? a.fit[x] : my_fit;
    my_fit_rows = c == x ? a.fit_rows[x] : my_fit_rows;
  }
  const uint32_t spare = present - 1u;                   // every class but one may end with a partly filled task
  const uint32_t even = a.waves > spare ? a.waves - spare : 1u;
  const uint32_t first = divide_up(sum - spare, k == 0u ? even : room);
  const uint32_t share = a.waves > spare ? higher(1u, wave.value(first, 0u)) : ~0u;
  const uint32_t least = wave.value(first, 4u) + spare;
  // candidates: one turn of even tasks, of as many rows as `rows`; any number of turns of the longest tasks; and how many turns even ones take
  const uint32_t own = k == 0u ? lower(share, my_fit_rows) : k == 1u ? my_fit_rows : k == 2u ? my_fit : a.waves;
  uint32_t tasks = divide_up(k < 3u ? my_units : least, own), step = own * my_unit;
  const uint32_t total = wave.quad_sum(tasks);
  uint32_t best = 0u;
  if (share > most && wave.value(total, 0u) > a.waves) {
    const uint32_t turns = wave.value(tasks, 12u);
    best = wave.value(total, 4u) <= a.waves ? 4u : 8u;
    if (best == 8u && turns <= 3u && room >= 3u) {
      const uint32_t shorter = higher(1u, divide_up(sum - spare, turns * a.waves - spare));
      tasks = divide_up(my_units, shorter);
      step = shorter * my_unit;
    }
  }
  TaskCut cut;
#pragma unroll
  for (uint32_t x = 0; x < 4u; ++x) {
    cut.tasks[x] = wave.value(tasks, best + x);
    cut.step[x] = wave.value(step, best + x);
  }
  return cut;
}

}  // namespace qkv
