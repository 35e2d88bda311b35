// Goes through attention's cut (paper_2605_03884_amd/csrc/attend_cut.h) for random shapes and class counts on the host; built and run by
// tests/test_attend_cut.py.  The device code is the one that is run: a wave's lanes are taken one after the other, and again until every
// value that a lane asks another one for is known.
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2605_03884_amd/csrc/attend_cut.h"

namespace {

struct Shape { uint32_t rows, chunk, waves, unit[4], fit[4], fit_rows[4]; };
struct Counts { uint32_t n[4]; };

struct Exchange {
  std::vector<std::array<uint32_t, 16>>& said;         // per exchange, what every lane put in
  size_t known, call;
  uint32_t lane;
  size_t put(uint32_t v) {
    if (call == said.size()) said.emplace_back();
    said[call][lane] = v;
    return call++;
  }
  uint32_t value(uint32_t v, uint32_t from) { const size_t i = put(v); return i < known ? said[i][from] : 64u; }
  uint32_t quad_sum(uint32_t v) {
    const size_t i = put(v);
    const uint32_t q = lane & ~3u;
    return i < known ? said[i][q] + said[i][q + 1] + said[i][q + 2] + said[i][q + 3] : 64u;
  }
};

template <int DS, bool KC>
qkv::TaskCut cut(const Shape& a, const Counts& g, bool& same) {
  std::vector<std::array<uint32_t, 16>> said;
  for (size_t known = 0;; ++known) {
    std::array<qkv::TaskCut, 16> out;
    size_t calls = 0;
    for (uint32_t lane = 0; lane < 16; ++lane) {
      Exchange e{said, known, 0, lane};
      out[lane] = qkv::cut_tasks<DS, KC>(a, g, lane, e);
      calls = e.call;
    }
    if (calls > known) continue;
    same = true;
    for (const auto& o : out)
      for (int c = 0; c < 4; ++c) same = same && o.tasks[c] == out[0].tasks[c] && o.step[c] == out[0].step[c];
    return out[0];
  }
}

constexpr uint32_t kGroup[3][4] = {{64, 64, 32, 32}, {64, 48, 32, 16}, {32, 32, 16, 16}};      // rows whose loads are in flight together (Prefetch)

}  // namespace

int main(int argc, char** argv) {
  const long cases = argc > 1 ? std::atol(argv[1]) : 1000;
  std::mt19937_64 rng(argc > 2 ? std::atol(argv[2]) : 1);
  const auto pick = [&](uint64_t n) { return rng() % n; };
  const auto logarithmic = [&](double lo, double hi) { return (uint32_t)std::lround(std::exp(std::log(lo) + (std::log(hi) - std::log(lo)) * (double)(rng() >> 11) / 9007199254740992.0)); };
  long several = 0, single = 0, longest = 0, finer = 0;
  for (long i = 0; i < cases; ++i) {
    const uint32_t di = (uint32_t)pick(3), D = 64u << di, rep = 1u + (uint32_t)pick(16);
    const uint64_t pairs = pick(2) ? logarithmic(1, 3000) : (uint64_t)(1u + pick(80)) * (1u << pick(4));
    const bool kc = di < 2 && pick(4) == 0;
    uint32_t T = logarithmic(1, pick(8) ? 30000 : 400000);
    if (pick(3) == 0) T = (T + 63u) / 64u * 64u + (uint32_t)pick(3) - 1u;
    if (kc) T = std::max(64u, T / 64u * 64u);
    if (kc && D == 128u && pick(2)) T += 32u;
    Counts g{};
    if (kc || pick(4) == 0) {
      g.n[pick(kc ? 3 : 4)] = T;
    } else {                                             // one to four classes, some of them nearly empty
      uint32_t left = T;
      const uint32_t last = (uint32_t)pick(4);
      for (uint32_t c = 0; c < 4; ++c)
        if (c != last && pick(3)) { g.n[c] = pick(4) ? (uint32_t)pick(left + 1u) : std::min(left, (uint32_t)pick(4)); left -= g.n[c]; }
      g.n[last] += left;
    }
    Shape a{};
    uint32_t rows = 0, least = 0;
    qkv::attend_plan(T, rep, pairs, &rows, &least);
    const uint32_t best = qkv::attend_more_tasks(T, rep, pairs, D, least);
    const uint64_t per = pairs * rep * (D + 2u);
    const uint64_t floats = per * (pick(2) ? best : least + pick(best - least + 1u)) + 4u;
    const uint32_t partials = qkv::cut_parameters(a, T, rep, pairs, D, kc, floats);
    bool same = false;
    const qkv::TaskCut k = kc ? (di == 0 ? cut<2, true>(a, g, same) : cut<4, true>(a, g, same))
                              : di == 0 ? cut<2, false>(a, g, same) : di == 1 ? cut<4, false>(a, g, same) : cut<8, false>(a, g, same);
    const uint32_t tasks = k.tasks[0] + k.tasks[1] + k.tasks[2] + k.tasks[3];
    const char* wrong = !same ? "lanes disagree" : nullptr;
    const bool turns = !kc && a.waves < partials;          // the kernel whose waves take several tasks
    if (!turns && tasks > a.waves) wrong = "a task without a wave";
    if (a.waves < 1u || a.waves > partials || per * partials + 4u > floats) wrong = "partials beyond the workspace";
    if (a.chunk * ((rep + 3u) & ~3u) > qkv::kLdsFloatsPerWave) wrong = "scores beyond LDS";
    for (int c = 0; c < 4; ++c) {
      if (g.n[c] == 0u) { if (k.tasks[c] != 0u) wrong = "a task of an absent class"; continue; }
      if (k.step[c] > a.chunk || k.step[c] == 0u) wrong = "a task longer than LDS holds";
      if (k.step[c] % a.unit[c] != 0u || a.unit[c] % kGroup[di][c] != 0u || (kc && k.step[c] % 32u != 0u)) wrong = "a task that is no whole number of groups";
      if ((uint64_t)k.tasks[c] * k.step[c] < g.n[c] || (uint64_t)(k.tasks[c] - 1u) * k.step[c] >= g.n[c]) wrong = "rows left out, or an empty task";
    }
    uint32_t cls = 0, at = 0, tau = 0;
    for (; tau < tasks && !wrong; ++tau) {                 // what waves ask for: every row once, in order
      uint32_t j0 = 0, j1 = 0;
      const int c = k.find(g, tau, j0, j1);
      while (cls < 4u && at == g.n[cls]) { ++cls; at = 0; }
      if (c != (int)cls || j0 != at || j1 <= j0 || j1 > g.n[cls]) wrong = "rows out of order";
      at = j1;
    }
    while (cls < 4u && at == g.n[cls]) { ++cls; at = 0; }
    uint32_t j0, j1;
    if (!wrong && (cls != 4u || k.find(g, tasks, j0, j1) != -1)) wrong = "rows left out";
    if (wrong) {
      std::printf("%s: D %u, %u heads, %llu pairs, %u tokens (%u %u %u %u), kc %d, %u waves, %u partials, tasks %u %u %u %u of %u %u %u %u rows\n", wrong, D, rep,
                  (unsigned long long)pairs, T, g.n[0], g.n[1], g.n[2], g.n[3], (int)kc, a.waves, partials, k.tasks[0], k.tasks[1], k.tasks[2], k.tasks[3],
                  k.step[0], k.step[1], k.step[2], k.step[3]);
      return 1;
    }
    several += turns && tasks > a.waves;
    single += !turns;
    finer += partials > least;
    longest += !turns && a.rows == 64u && k.step[1] > 64u && g.n[1] != 0u;
  }
  std::printf("cut ok: %ld cases, %ld with several tasks a wave, %ld with one, %ld finer, %ld longest of LDS\n", cases, several, single, finer, longest);
  return several && single && finer && longest ? 0 : 2;
}
