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
  int ranges;       // key ranges per query block: 1, 2, 4 or 8
  int rotation;     // work-groups in flight per XCD, or 0: every list is walked from its head
  int group_rows;   // query rows of a work-group: the block size, or 64 or 128 for the dense call
  int spread_bits;  // log2 of the XCDs that share a (head, range) pair
  int64_t grid;     // work-groups launched
};

// Rows of a work-group.  The dense call, whose rows all see the same keys, takes
// 128-row groups, but 64 rows where those would be so few that most CUs stay
// idle (1,056 queries of one head: 13.8 us against 15.9), or would pad a
// short query sequence by more than a tenth (774 queries of 10 heads: 154 and 158).
inline int attn_group_rows(int64_t bh, int64_t lq, int block, bool dense, int ranges) {
  if (!dense) return block;
  const int64_t wide = (lq + 127) / 128, narrow = (lq + 63) / 64, n_wide = wide * bh * ranges;
  return n_wide <= 64 || (n_wide > 256 && 20 * wide > 11 * narrow) ? 64 : 128;
}

// How many XCDs share a (head, range) pair.  One keeps the pair's K/V in one
// L2, but an XCD with only a few pairs runs as long as its heads' lists are
// (per-head budgets differ).  So a pair is shared until each XCD has four
// units, as long as a unit keeps 4,096 query rows (half of what an XCD holds):
// 8 heads with budgets from 0.5 to 1.5 of the mean, 21,332 queries, took
// 0.56 ms shared by four and 0.71 unshared; 6,413 queries 0.62 and 0.44.  The
// units of all pairs have to deal out evenly in any case, but a pair is never
// shared by more XCDs than it has groups: the work-groups of the empty units
// return at once, yet count as placed when the dispatcher goes round the CUs
// (dense call, 35 heads of 200 queries, two groups each: 21.5 us shared by
// eight, 16.4 by one or two), and eight times as many work-groups as items can
// pass the launch limit of 2^32 threads.
inline int attn_spread_bits(int64_t pairs, int64_t groups, int group_rows) {
  auto enough = [&](int bits) {
    const int64_t units = pairs << bits;
    return units % 8 == 0 && (units >= 32 || ((groups * group_rows) >> (bits + 1)) < 4096);
  };
  int bits = 0;
  while (bits < 3 && (int64_t(1) << bits) < groups && !enough(bits)) ++bits;
  return bits;
}

// Work-groups launched: whole rounds of eight units (one per XCD), each of the
// groups a unit can hold.  The kernel's decode of blockIdx matches.
inline int64_t attn_grid(int64_t pairs, int64_t groups, int bits) {
  const int64_t units = ((pairs << bits) + 7) / 8 * 8;
  return units * ((groups + (1 << bits) - 1) >> bits);
}

// The number of key ranges R (1, 2, 4 or 8) that minimises an estimate of the
// call's time, in units of one 32-key tile step with the chip full:
//   - an item (one query block and range) takes its share of the list plus about
//     16 steps of fixed work (list scan, Q, first tiles, epilogue) and, with
//     R > 1, 3 for its partial result and the merge (twice as many steps at
//     D = 64, whose step is half as long);
//   - the chip holds 65,536 query rows at D = 128, 98,304 at D = 64 (two, three
//     waves per SIMD): x rounds of items.  A partly filled last round takes half
//     an item's time when nearly empty, since the waves left share less;
//   - K and V of one range beyond about 20 MB lose the L2's reuse between the
//     items in flight (15%, and 30% more beyond 40 MB).
// A range keeps at least 256 listed keys.  Against the best R of a sweep over 25
// shapes (1 to 24 heads, 512 to 72,000 queries, 1,152 to 144,512 keys, both
// head dims and block sizes, sparse and dense) the estimate's choice is 0.2%
// slower on average and 1.4% at worst; 16 ranges were never the best.
// The estimate reads the list length, not the kind of call, so that the dense
// call and a sparse call whose lists can name every block are cut alike.
// With several ranges the lists are rotated (attn_fwd.hip) where some cannot name
// every block and at least eight rounds of items let the work-groups in flight
// spread out in time (mid-scale call, 11,520 queries: 3.25 ms rotated and 4.01
// plain at 17 rounds; 6,413 queries and 8 heads: 478 and 476 us at 3).
inline AttnPlan attn_plan(int64_t bh, int64_t lq, int64_t lk, int d, int block, int64_t kv_stride, bool dense,
                          bool may_split) {
  const int64_t nq = (lq + block - 1) / block, nk = (lk + block - 1) / block;
  // the dense call lists every key block, so it takes the ranges of a full list
  const int64_t list_blocks = dense || kv_stride > nk ? nk : kv_stride;
  const double list_keys = double(list_blocks) * block;
  const double rows = double(bh) * double(nq) * block;
  const double rows_held = 32768.0 * attn_waves_per_simd(d);
  const double kv_bytes = double(lk) * 4.0 * d;
  AttnPlan plan{1, 0, 0, 0, 0};
  double best = 0.0, best_rounds = 0.0;
  for (int r = 1; r <= 8; r *= 2) {
    if (r > 1 && (!may_split || list_keys < 256.0 * r)) break;
    const double rounds = rows * r / rows_held, whole = floor(rounds), part = rounds - whole;
    const double item = list_keys / 32.0 / r + (r > 1 ? 19.0 : 16.0) * (128.0 / d);
    double t = item * (whole + (part > 0.0 ? 0.5 + 0.5 * part : 0.0));
    if (rounds > 1.0) {
      if (kv_bytes / r > double(20 << 20)) t *= 1.15;
      if (kv_bytes / r > double(40 << 20)) t *= 1.3;
    }
    if (r == 1 || t < best) {
      best = t;
      best_rounds = rounds;
      plan.ranges = r;
    }
  }
  if (plan.ranges > 1 && list_blocks < nk && best_rounds >= 8.0) plan.rotation = int(rows_held) / 8 / block;
  plan.group_rows = attn_group_rows(bh, lq, block, dense, plan.ranges);
  const int64_t groups = (lq + plan.group_rows - 1) / plan.group_rows, pairs = bh * plan.ranges;
  plan.spread_bits = attn_spread_bits(pairs, groups, plan.group_rows);
  plan.grid = attn_grid(pairs, groups, plan.spread_bits);
  return plan;
}

}  // namespace sparstar
