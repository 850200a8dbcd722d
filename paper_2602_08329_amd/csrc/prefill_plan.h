// How a prefill launch divides its prompts: the waves and key sides of a
// workgroup, its block of queries, and the order of the blocks.  Host code (and
// the block order, which the kernel shares), without device calls.
#pragma once

#include <math.h>

#include <algorithm>

#include "prhs_internal.h"

namespace prhs {

// Waves of a workgroup: two or three a SIMD, as many as their registers allow.
constexpr int waves_of(int w) { return w == 32 ? 8 : 12; }
// A second workgroup on the CU: at d 64, where 128 registers a wave do without
// scratch (126 with 8 spilled for the paged one-sided form: 2 us more a launch).
constexpr bool two_per_cu(int d, int w, int ns, bool paged) { return d == 64 && w == 32 && (ns == 1 ? !paged : ns == 4 && paged); }
constexpr int waves_per_simd(int d, int w, int ns, bool paged) {
  return (two_per_cu(d, w, ns, paged) ? 2 : 1) * waves_of(w) / 4;
}
constexpr int kQueries = 256;    // queries per workgroup of 32-query waves with one key side
constexpr int kPackBlocks = 48;  // blocks a unit up to which a launch's packing is worked out
constexpr int kXcds = 8;         // accelerator dies, each with its own L2
// Units of an XCD (`per` of them, nqb blocks each) that it works through side by
// side, longest blocks first over all of them: a launch ends with the last
// group's blocks, so a group has at least kGroupRounds rounds of blocks for the
// XCD's CUs, and no more, as its units' K and V share one L2 (d 128, us, with
// groups of 1 | 2 | 4 | all units: 64 units x 1900 170 | 143 | 108 | 106, 40 x
// 2221 129 | 138 | 135 | 88 (5 an XCD), 96 x 2124 224 | 216 | 211 | 188, 32 x
// 7490 718 | 674 | 652 | 653, 160 x 14310 11790 | 11590 | 11610 | 12890).  Groups
// are of equal size but for the last.
constexpr int kGroupRounds = 4;
inline int unit_group(int per, int nqb, int cus) {
  const int least = (kGroupRounds * (cus > 0 ? cus : 256) / kXcds + nqb - 1) / nqb;
  const int groups = std::max(1, per / std::max(1, least));
  return std::max(1, (per + groups - 1) / groups);
}

// Query block and (batch, head) unit of workgroup L.  Workgroups go to the 8
// XCDs round-robin by id.  When the units divide over the XCDs, XCD x works
// through its own units in groups of `group`, within a group longest blocks
// first over all of its units: a unit's K and V stay in one L2, its blocks run
// side by side, and the launch ends with the short blocks.  Otherwise all units
// form one group over all XCDs (44 units x 8245 at d 128 1108 us; a unit's
// blocks one after the other 1745).
__host__ __device__ __forceinline__ void block_of(int units, int nqb, int group, int L, int* bh, int* qb) {
  if (units % kXcds == 0) {
    const int per = units / kXcds, x = L % kXcds, i = L / kXcds;
    const int grp = i / (group * nqb), j = i - grp * (group * nqb);
    const int left = per - grp * group, gu = left < group ? left : group;
    *bh = x * per + grp * group + j % gu;
    *qb = nqb - 1 - j / gu;
  } else {
    *bh = L % units;
    *qb = nqb - 1 - L / units;
  }
}

// Time of a launch of `units` blocks of each of the n costs on `slots` places
// for one block at a time, each block to the place that is free first: places
// as groups of equal load, of which each cost splits at most one.
inline float packed_time(const float* cost, int n, long long units, long long slots) {
  struct Group {
    float load;
    long long count;
  };
  Group g[kPackBlocks + 1];
  int m = 1;
  g[0] = {0.f, slots};
  for (int i = 0; i < n; ++i) {
    for (long long left = units; left > 0;) {
      int lo = 0;
      for (int j = 1; j < m; ++j) lo = g[j].load < g[lo].load ? j : lo;
      const long long take = std::min(left, g[lo].count);
      left -= take;
      if (take == g[lo].count) {
        g[lo].load += cost[i];
      } else {
        g[lo].count -= take;
        g[m++] = {g[lo].load + cost[i], take};
      }
    }
  }
  float t = 0.f;
  for (int j = 0; j < m; ++j) t = std::max(t, g[j].load);
  return t;
}

// What a plan depends on: the prompt's queries T, the head dimension, the cache
// layout and the window (psaw_f and sink of Eq. psaw where psaw is nonzero).
struct PrefillShape {
  int T, d, paged, psaw;
  double psaw_f;
  int sink;
};

// How a launch divides its units: waves of w queries, ns key sides, blocks of
// qblock queries, the first of qfirst.
struct PrefillPlan {
  int w, ns, qblock, qfirst;
  int blocks(int T) const { return 1 + (std::max(T - qfirst, 0) + qblock - 1) / qblock; }
};

// The plan of least time, its blocks packed on the CUs.  A block costs
// `step` for each of its key tiles (64, 64, 128 and 128 keys) and `fixed`
// once (for a prompt of T tokens), in us; a step costs by the waves that share a
// SIMD, as it is their issue and the chain of one wave that it waits for.
// Fitted to 2600 timed launches (within 6% on average; the plan taken is 2% from
// the best of its launch).  What each is for, d 128, in us, with (16 queries, one
// side | 32 queries, one | two | four sides):
//   256 queries fill the LDS reads best, on launches of many blocks: 32 heads
//   x 4096 - | 187 | 216 | 273, 128 x 450 33.2 | 30.1 | 36.2 | 47.7;
//   sides shorten the longest block of few units: 32 x 537 20.8 | 23.6 | 20.6
//   | 17.6, 4 x 8000 - | 279 | 171 | 123;
//   three narrow waves a SIMD hide a chain that two leave bare, where a CU
//   gets about one block: 128 x 265 15.6 | 16.8 | 22.9 | 27.2, 128 x 173 11.6
//   | 12.9 | 13.0 | 20.5, 16 x 6000 213 | 228 | - | -.
// The first block may differ from the others, and the last be short: it sees
// the most keys (256 x 536 at 32 queries 68.2 with even blocks, 64.4 with 128
// first and then 256; 128 x 316 at 16 queries 19.0 even, 17.9 with 192 first).
// Prompts of more than kShortBlocks blocks put what is left over in the last (8 x
// 12197 at 16 queries 433, in the first 466).  At d 64 a second workgroup of the
// wide waves fits a CU where 128 registers hold them: 256 x 1024 99 -> 79, 64 x
// 7777 834 -> 731.
// Every layer of a model asks for its plan, so its work is bounded: prompts of
// more than kPackBlocks blocks are summed over that many of them, and a form is
// packed only where an even spread of its blocks would win (on one CPU, us: 40
// units x 2000 17.8 -> 2.6, 32 x 4096 5.3 -> 2.4, one unit x 131072 79 -> 1.3).
constexpr int kShortBlocks = 16;
// Key sides on launches of more than two rounds of blocks take longer than the sum
// of their blocks (d 128, 8 units x 11000 362 us by the sum, 400 timed, 16
// queries 359; under a window 8 x 10611 287, 319 and 285).
constexpr float kSidesLate = 1.05f;
inline PrefillPlan plan_of(const PrefillShape& s, long long units, int cus) {
  const int T = s.T, d = s.d;
  const bool paged = s.paged != 0;
  const auto whole = [](int q, int w) { return (q + w - 1) / w * w; };
  const int nwide = (T + kQueries - 1) / kQueries;
  if (cus <= 0 || nwide * units >= 8LL * cus)
    return {32, 1, kQueries, whole(T - (nwide - 1) * kQueries, 32)};
  // one block, one tile or two: the wave's chain is all there is (64 x 113 8.4
  // with 16 queries, 8.8, 10.0 and 8.7)
  if (d == 128 && T <= 128 && units <= cus) return {16, 1, whole(T, 16), whole(T, 16)};
  struct Cost {
    float step[3], fixed;
  };
  // d 128, d 64, d 64 paged; the last of each is the one that shares a CU,
  // where the launch has more blocks than CUs
  static const Cost costs[3][5] = {
      {{{1.27f, 1.62f, 2.12f}, 6.17f}, {{2.03f, 2.65f}, 5.80f}, {{1.86f, 2.92f}, 7.54f}, {{0.92f, 1.70f}, 7.43f}, {}},
      {{{1.40f, 1.47f, 1.72f}, 3.95f}, {{1.67f, 2.00f}, 3.91f}, {{1.59f, 2.25f}, 4.86f}, {{0.56f, 1.19f}, 4.65f},
       {{1.65f, 2.80f}, 6.94f}},
      {{{1.04f, 1.47f, 1.68f}, 4.65f}, {{1.74f, 2.08f}, 4.73f}, {{1.66f, 2.20f}, 5.81f}, {{1.36f, 1.62f}, 5.34f},
       {{1.18f, 1.80f}, 6.94f}}};
  const Cost* const table = costs[d == 128 ? 0 : paged ? 2 : 1];
  PrefillPlan best = {32, 1, kQueries, kQueries};
  float least = INFINITY;
  for (int v = 0; v < 4; ++v) {
    const int w = v == 0 ? 16 : 32, ns = v == 0 ? 1 : 1 << (v - 1), kt_log2 = v < 2 ? 6 : 7;
    const auto tiles_of = [&](int keys) { return (keys + (1 << kt_log2) - 1) >> kt_log2; };
    const int most = w * waves_of(w) / ns, nmin = (T + most - 1) / most;
    const int sizes[4] = {whole((T + nmin - 1) / nmin, w), whole((T + nmin) / (nmin + 1), w), most,
                          v == 3 ? most : most / 2};
    // each size with what is left over in the first block, then in the last
    for (int k = nmin > kShortBlocks ? 5 : 0; k < (nmin > kShortBlocks ? 6 : 8); ++k) {
      const int qb = sizes[k / 2];
      const int n = k % 2 ? (T + qb - 1) / qb : 1 + (std::max(T - most, 0) + qb - 1) / qb;
      const int qf = k % 2 ? qb : std::min(most, whole(T - (n - 1) * qb, w));
      const bool shared = two_per_cu(d, w, ns, paged) && n * units > cus;
      const Cost& c = table[shared ? 4 : v];
      const long long slots = shared ? 2LL * cus : cus;
      const auto time_of = [&](int j) {
        const int end = std::min(T, qf + j * qb), q0 = j ? qf + (j - 1) * qb : 0;
        int tiles = tiles_of(end);
        if (s.psaw) {
          const int nsink = tiles_of(std::min(s.sink, end));
          const int first = psaw_first_visible(s.psaw_f, s.sink, q0 + 1);
          tiles = std::min(tiles, nsink + std::max(tiles - std::max(first >> kt_log2, nsink), 0));
        }
        const int waves = (end - q0 + w - 1) / w * ns;
        return c.step[(waves + 3) / 4 - 1] * (float)tiles + c.fixed;
      };
      float cost[kPackBlocks], sum = 0.f, longest = 0.f;
      if (n <= kPackBlocks) {
        for (int j = n - 1; j >= 0; --j) {  // longest first
          const float t = cost[n - 1 - j] = time_of(j);
          sum += t;
          longest = std::max(longest, t);
        }
      } else {  // every skip-th block, from the middle of the first skip; the last may be short
        const int skip = (n + kPackBlocks - 1) / kPackBlocks;
        int m = 0;
        for (int j = skip / 2; j < n; j += skip, ++m) sum += time_of(j);
        sum *= (float)n / (float)m;
        longest = std::max(time_of(n - 1), time_of(n - 2));
      }
      // no packing is shorter than an even spread, and many blocks pack evenly
      const float more = ns > 1 && n * units > 2 * slots ? kSidesLate : 1.f;
      float t = more * std::max(longest, sum * (float)units / (float)slots);
      if (t < least && n <= kPackBlocks) t = more * packed_time(cost, n, units, slots);
      if (t < least) least = t, best = {w, ns, qb, qf};
    }
  }
  return best;
}

}  // namespace prhs
