// How an attention call is cut up (host code): key ranges per query block, the
// rows of a work-group, the XCDs that share a (head, range) pair, and whether
// the lists are walked from a rotated start.  The kernel (attn_fwd.hip) takes
// the cut through AttnArgs.
#pragma once

#include <math.h>
#include <stdint.h>

#include "launch.h"

namespace sparstar {

struct AttnPlan {
  int ranges;       // key ranges per query block: 1, 2, 4, 8 or 16
  int rotation;     // work-groups in flight per XCD, or 0: every list is walked from its head
  int group_rows;   // query rows of a work-group: the block size, or 64 or 128 for the dense call
  int spread_bits;  // log2 of the XCDs that share a (head, range) pair
  int64_t grid;     // work-groups launched
};

// How many XCDs share a (head, range) pair.  One keeps the pair's K/V in one
// L2, but an XCD with only a few pairs runs as long as its heads' lists are
// (per-head budgets differ).  So a pair is shared until each XCD has four
// units, as long as a unit keeps 3,300 query rows (two fifths of what an XCD
// holds): 8 heads with budgets from 0.5 to 1.5 of the mean, 21,332 queries, took
// 0.56 ms shared by four and 0.71 unshared; 6,413 queries 0.62 and 0.44; two
// heads of such budgets, 26,971 queries, 0.85 ms shared by four and 0.67 by
// eight (0.61 and 0.72 with equal budgets).  262 shapes timed with every
// sharing took 3.3% more than with the best one where budgets are equal and 3.8%
// where they differ; at 4,096 rows 3.2% and 4.9%, shared by eight throughout
// 6% and 7%.  The units of all pairs have to deal out evenly in any case: up to a
// sixth of the last round of units empty gains where K/V exceed the L2 (23
// heads, 3,152 queries, 28,266 keys: 628 us shared by eight, 401 unshared), but
// costs 5 to 10% where they don't.
//
// Sharing by two or four leaves empty work-groups at the end of the units.  They
// return at once, yet count as placed when the dispatcher goes round the CUs, so
// where they would be more than a sixteenth of the items the pairs are shared by
// eight, which needs none.  19 heads of 13 groups, about one work-group per CU:
// 71.1 us with a fifth of the work-groups empty, 56.2 without; 25 heads of 9 30.8 and
// 21.8.
inline int attn_spread_bits(int64_t pairs, int64_t groups, int group_rows) {
  auto enough = [&](int bits) {
    const int64_t units = pairs << bits, empty = units * ((groups + (1 << bits) - 1) >> bits) - pairs * groups;
    return units % 8 == 0 && 16 * empty <= pairs * groups &&
           (units >= 32 || ((groups * group_rows) >> (bits + 1)) < 3300);
  };
  int bits = 0;
  while (bits < 3 && !enough(bits)) ++bits;
  return bits;
}

// Work-groups launched: every item, or the groups that whole units can hold.
// The kernel's decode of blockIdx matches.
inline int64_t attn_grid(int64_t pairs, int64_t groups, int bits) {
  return bits == 3 ? pairs * groups : (pairs << bits) * ((groups + (1 << bits) - 1) >> bits);
}

// An estimate of a call's time in microseconds, for one cut of it.  rho is the
// share of the key blocks that a list can name (1 for the dense call).
//
// What it counts, on the XCD with the most work-groups:
//   - tile steps: a work-group walks its share of the list, plus some 4 steps of
//     fixed work and, on sparse lists cut into ranges, the 1.93 standard deviations by
//     which the longest share exceeds the mean.  A step's time depends on how
//     many work-groups share the CU (kStepUs, D and waves per work-group); whole
//     rounds run full, the last one with what is left of it;
//   - K/V from beyond the L2: once per round for what the lists cover of the
//     range, and for every work-group where those in flight are too far apart for
//     the L2 (1.7 MB of it): by a little of the random spread of their positions
//     in the range, by a quarter of the range per round that they drift without
//     rotation, by 9% of it with rotation;
//   - the merge of the partial results.
// The constants are fitted to some 2,000 random shapes, each timed at every cut (1
// to 200 heads, 64 to 72,000 queries, 1,100 to a million keys, 3% to 95% density
// and dense, uniform and clustered lists, both head dims and block sizes), and to
// 68 large ones (8 and 24 heads, 25,920 to 72,000 queries, 10% to 80%, budgets
// equal and per head).  The chosen cut is 0.8% slower than the best one on average
// (13% in one shape of a hundred), and on the large ones (6% at most).  A count of
// ranges from tile steps and K/V per range alone, of at most 8, lost 13%: it took
// 257 us for 1,000 queries of one head over 144,000 keys (16 ranges: 150), and
// two ranges for short lists, where the merge costs more than it saves (7,686
// queries of 4 heads, lists of 7 blocks of 128: 35 us, one range 23).
inline double attn_time_us(int64_t bh, int64_t lq, int64_t lk, int d, int block, double rho, bool dense, int ranges,
                           bool rotated, int group_rows) {
  // by work-groups per CU, for work-groups of two and of four waves
  static constexpr double kStepUs128[2][4] = {{.44, .67, .69, .87}, {.48, .76}};
  static constexpr double kStepUs64[2][4] = {{.63, .83, .97, 1.07}, {.67, .97}};
  const int waves = group_rows / 32;
  const double* step_us = (d == 64 ? kStepUs64 : kStepUs128)[waves / 4];
  const int per_cu = 4 * kAttnWavesPerSimd / waves;
  const double held = 32.0 * per_cu;  // work-groups an XCD holds
  const int64_t groups = (lq + group_rows - 1) / group_rows, pairs = bh * ranges;
  const int bits = attn_spread_bits(pairs, groups, group_rows);
  const double units = double(((pairs << bits) + 7) / 8);                    // per XCD
  const double unit_groups = double((groups + (1 << bits) - 1) >> bits);
  const double work_groups = bits == 3 ? double((pairs * groups + 7) / 8) : units * unit_groups;
  const double rounds = work_groups / held;
  const double whole = floor(rounds), part = rounds - whole;

  const double sub = double(block) / attn_tile_keys(d);
  const double list_blocks = rho * double((lk + block - 1) / block) / ranges;
  const double steps = list_blocks * sub + (d == 64 ? 3.7 : 4.5);
  const double deviation = sqrt(list_blocks * (1.0 - rho));  // of a share's entries
  const double longest = steps + (ranges > 1 && !dense ? 1.93 * deviation * sub : 0.0);
  double t = 2.3 + whole * steps * step_us[per_cu - 1];
  if (part > 0.0) t += longest * step_us[int(fmax(1.0, ceil(part * per_cu - 1e-9))) - 1];
  else t += (longest - steps) * step_us[per_cu - 1];

  const double token_bytes = 4.0 * d, range_bytes = double(lk) * token_bytes / ranges;
  double apart = 0.12 * deviation / rho * block * token_bytes;
  if (!dense && rounds > 1.0) apart += (rotated ? 0.09 : 0.25 * fmin(1.0, rounds - 1.0)) * range_bytes;
  apart = fmin(apart, range_bytes);
  const double miss = apart > 1.7e6 ? 1.0 - 1.7e6 / apart : 0.0;
  const double covered = dense ? 1.0 : 1.0 - pow(1.0 - rho, fmin(unit_groups, held));
  const double every = work_groups * list_blocks * block * token_bytes;
  const double once = fmin(every, units * fmax(1.0, unit_groups / held) * range_bytes * covered);
  t += (once * (1.0 - miss) + every * miss) / 4.7e6;
  if (ranges > 1)
    t += 3.7 + 0.25 * ranges * block * d / 8192.0 + double(bh) * double(lq) * ranges * token_bytes / 6.3e6;
  return t;
}

// The cut with the least estimated time.  The dense call's work-groups take 64 or
// 128 rows: 128 feed twice the queries per K/V byte loaded, 64 fill more CUs and
// pad less.  With several ranges the lists are rotated (attn_fwd.hip) where the
// estimate says so.  A sparse call whose rows can name every block takes the
// ranges of the dense call, so that full lists give the dense call's bits; what
// its lists hold is not known here, and from eight rounds of work-groups on it
// is rotated (the kernel leaves the lists that are full plain): lists of 25% in
// rows of full width, 24 heads, 72,000 queries, 144,512 keys, took 50.4 ms in 4
// plain ranges and take 32.4, as in rows of their own width; 11,520 queries 3.78
// and 3.17.  Rotated lists do better in narrow ranges (35.5 ms in 2), so of two
// cuts of full rows that differ by less than 0.6% the one with more ranges is taken.
inline AttnPlan attn_plan(int64_t bh, int64_t lq, int64_t lk, int d, int block, int64_t kv_stride, bool dense,
                          bool may_split) {
  const int64_t nk = (lk + block - 1) / block;
  const bool full = dense || kv_stride >= nk;
  const double rho = full ? 1.0 : double(kv_stride) / double(nk);
  AttnPlan plan{1, 0, 0, 0, 0};
  double best = 0.0;
  for (int rows = full ? 64 : block; rows <= (full ? 128 : block); rows *= 2)
    for (int r = 1; r <= (may_split ? kSplits : 1); r *= 2) {
      const int64_t g = (lq + rows - 1) / rows;
      if (r > 1 && attn_grid(bh * r, g, attn_spread_bits(bh * r, g, rows)) * 2 * rows >> 32) break;  // launch limit
      // (rotation only matters where the work-groups don't all start at once)
      const bool rounds = bh * r * g * rows > 32768 * kAttnWavesPerSimd;
      for (int rotated = 0; rotated <= (r > 1 && !full && rounds); ++rotated) {
        const double t = attn_time_us(bh, lq, lk, d, block, rho, full, r, rotated, rows);
        if (plan.group_rows == 0 || t < (full && r > plan.ranges ? 1.006 * best : best)) {
          best = plan.group_rows == 0 ? t : fmin(best, t);
          plan.group_rows = rows;
          plan.ranges = r;
          plan.rotation = rotated ? 32 * 4 * kAttnWavesPerSimd / (rows / 32) : 0;
        }
      }
    }
  if (!dense) plan.group_rows = block;
  const int64_t groups = (lq + plan.group_rows - 1) / plan.group_rows, pairs = bh * plan.ranges;
  const int64_t held = 32 * 4 * kAttnWavesPerSimd / (plan.group_rows / 32);  // work-groups an XCD holds
  if (full && !dense && plan.ranges > 1 && pairs * groups >= 8 * 8 * held) plan.rotation = int(held);
  plan.spread_bits = attn_spread_bits(pairs, groups, plan.group_rows);
  plan.grid = attn_grid(pairs, groups, plan.spread_bits);
  return plan;
}

}  // namespace sparstar
