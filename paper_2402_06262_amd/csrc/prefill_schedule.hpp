// How the matrix-core prefill passes cut a prompt into workgroups.  Host code, shared by the launchers and by the workspace
// query (a pass that several workgroups divide needs room for their partial sums).
//
// The units of one call are anything from one to tens of thousands, and a workgroup walks its tiles one after the other, about
// a microsecond each where it has a compute unit to itself.  With few units the length of that walk is the time of the pass, so
// a block of owned rows is divided further, in this order:
//   paired   a long and a short block of 128 owned rows per workgroup, equal work for all; several workgroups may take a share
//            each of the streamed tiles (split);
//   single   one block per workgroup, split likewise: half the walk for the same number of tiles per share;
//   parts    the four waves of a workgroup share 64 or 32 owned rows (see Shares in prefill_planes.hip).
// More shares are more workgroups for the rounds in which they fill the chip, the last of which may be nearly empty, against
// what a share costs by itself (its owned rows, its first tiles, its sums): six to eight tiles' time (`rounds_split`).
// Column pass, us, with two shares and 64 owned rows at most -> now:
//   1 unit  x 8 heads x 3852 tokens of fp32 / 128  823 -> 125     2 units x 8 x 4396 of bf16 / 64   178 -> 60
//   3 units x 8 heads x 515 tokens of bf16 / 128    73 -> 12      1 unit  x 4 x 426 of bf16 / 128    30 -> 8
// These rules count workgroups, and where workgroups are about as many as the chip holds a count says little: 24 units x 2500
// tokens of fp32 / 128 took 344 us where pairs in two shares take 270, 100 x <= 1500 of bf16 / 128 124 against 116.  So what they
// pick is held against the schedule of one or two shares that serves many units, by an estimate of both passes' time
// (`estimate`), and left where that is less.  Whole prompts against one or two shares everywhere: 240 of 1 to 1000 units geometric
// mean 1.49, lowest 0.96; 420 of bf16 / 128 1.36 and 0.92; 120 of groups of 9 to 40 heads 1.88 and 0.95.
#pragma once
#include "kernels.hpp"

#include <math.h>

namespace roco {

struct PassPlan {
  bool wide;   // bf16 / 128: the kernels of prefill_mfma.hip (256 owned rows, tile ring, software-pipelined)
  int parts;   // waves that share 32 owned rows: 1, 2 or 4
  int split;   // workgroups that share a block's streamed tiles
  int paired;  // 1: a long and a short block per workgroup
  int ids;     // workgroups per stream (a unit, or a unit's query head)
};

struct PlanRule {
  int resident;      // workgroups that run at a time, for rounds_split; 0: as many shares as bring paired_want workgroups
  int paired_want;   // workgroups that make pairs of blocks worth while
  int paired_tiles;  // ... the fewest tiles of a share of theirs
  int paired_split;  // ... and the most shares: beyond, single blocks of as many shares are twice the workgroups
  int single_want, single_tiles;  // the same for single blocks
  int most_parts;
};

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int power_of_two_from(int want, long long have) {  // smallest power of two that brings `have` to `want`
  int s = 1;
  while (s < 64 && have * s < want) s *= 2;
  return s;
}

// Rows of a streamed tile of the kernels in prefill_planes.hip; the general grouped column pass takes the smaller ones.
inline int planes_tile_rows(int dtype, int head_dim, int parts, bool small) {
  const int rows = head_dim == 128 && dtype == 0 ? 32 : dtype == 0 || small ? 64 : 128;
  return rows > 32 * parts ? rows : 32 * parts;
}
// Streamed tiles of a whole column pass for the first keys: with a group's heads inside a result tile, two times 16 / group
// query positions per 32 rows.
inline bool heads_in_tile(int group) { return (group >= 2 && group <= 8) || group == 16; }
inline int heads_one_by_one(int group) { return heads_in_tile(group) ? 1 : group; }
inline int column_tiles(int tile_rows, int group, int L_max) {
  if (heads_in_tile(group)) return ceil_div(L_max, tile_rows / 32 * 2 * (16 / group));
  return ceil_div(L_max, tile_rows) * group;
}

inline int rounds_split(long long workgroups, int resident, int tiles, double own_tiles, int most_split) {
  int split = 1;
  double least = 0.0;
  for (int s = 1; s <= most_split; s *= 2) {
    const long long rounds = (workgroups * s + resident - 1) / resident;
    const double time = (rounds + 0.3) * (static_cast<double>(tiles) / s + own_tiles);
    if (s == 1 || time < least) { least = time; split = s; }
  }
  return split;
}

// heads: of a tile position that is taken head by head (the general grouped column pass), else 1.  A share then consists of whole
// positions, and what a share costs by itself it costs for each of them: 64 units x 15 heads x 1000 tokens of fp32 / 128 were cut
// into eight shares, column pass 910 us against 815 in two; 16 x 9 x 300 of bf16 / 64 into sixteen of five positions, 27.2 against 23.3.
template <class TilesFn>
inline PassPlan plan_planes(long long streams, int L_max, const PlanRule& r, int most_split, int heads, TilesFn tiles) {
  const auto positions = [&](int parts) { return tiles(parts) / heads; };
  PassPlan p = {false, 1, 1, 1, ceil_div(ceil_div(L_max, 128), 2)};
  const long long pairs = streams * p.ids;
  p.split = r.resident != 0 ? rounds_split(pairs, r.resident, tiles(1), 6.0 * heads, most_split) : power_of_two_from(r.paired_want, pairs);
  if (p.split <= most_split && p.split <= r.paired_split && pairs * p.split >= r.paired_want && tiles(1) >= r.paired_tiles * p.split && p.split <= positions(1)) return p;
  long long best = 0;
  for (int parts = 1; parts <= r.most_parts; parts *= 2) {
    const int ids = ceil_div(L_max, 128 / parts);
    int split = power_of_two_from(r.single_want, streams * ids);
    while (split > 1 && (split > most_split || tiles(parts) < r.single_tiles * split || split > positions(parts))) split /= 2;
    const long long total = streams * ids * split;
    if (2 * total >= 3 * best) {  // more waves per block only where they bring half as many workgroups again
      best = total;
      p = {false, parts, split, 0, ids};
    }
    if (4 * total >= 3 * r.single_want) break;
  }
  return p;
}

// dtype 0 = fp32, 1 = bf16
inline PassPlan filling_rows(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
  const long long streams = static_cast<long long>(units) * group;
  if (dtype == 1 && head_dim == 128) {
    const int ids = ceil_div(ceil_div(L_max, 256), 2);
    if (L_max <= 512 && streams * ids >= 480) return {true, 1, 1, 1, ids};  // one block, or an even pair, per workgroup
    int split = power_of_two_from(480, streams * ids);
    while (split > most_split) split /= 2;
    if (streams * ids * split >= 200 && ceil_div(L_max, 64) >= 8 * split) return {true, 1, split, 1, ids};
  }
  const PlanRule r = dtype == 1 ? (head_dim == 64 ? PlanRule{0, 480, 2, 4, 480, 2, 4} : PlanRule{0, 384, 4, 4, 384, 3, 4})
                                : (head_dim == 64 ? PlanRule{768, 480, 2, 4, 1024, 3, 2} : PlanRule{512, 384, 6, 4, 384, 3, 1});
  return plan_planes(streams, L_max, r, most_split, 1,
                     [&](int parts) { return ceil_div(L_max, planes_tile_rows(dtype, head_dim, parts, false)); });
}

inline PassPlan filling_columns(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
  if (dtype == 1 && head_dim == 128 && L_max <= 512 && units >= 480) return {true, 1, 1, 1, 1};
  // 256 owned rows from four blocks on (three are an uneven pair), or two with several heads' tiles for each.  Whole prompts, us,
  // with 128 / 256: 512 units x 800 tokens 212 / 187, 256 x 1000 131 / 117, 100 x 4 heads x 700 160 / 147, 64 x 1000 59 / 60; of three
  // blocks 190 x 673 99.6 / 94.5, but prompts of up to 673 75.2 / 81.3, of up to 693 on 471 units 143 / 148, 130 x 640 62 / 66.
  if (dtype == 1 && head_dim == 128 && (L_max > 768 || (group > 1 && L_max > 512))) {
    const int ids = ceil_div(ceil_div(L_max, 256), 2), tiles = column_tiles(64, group, L_max);
    const int split = rounds_split(static_cast<long long>(units) * ids, 512, tiles, 8.0, most_split);
    if (static_cast<long long>(units) * ids * split >= 250 && tiles >= 6 * split) return {true, 1, split, 1, ids};
  }
  const PlanRule r = dtype == 1 ? (head_dim == 64 ? PlanRule{0, 1024, 4, 16, 1024, 2, 4} : PlanRule{0, 360, 4, 4, 480, 2, 4})
                                : (head_dim == 64 ? PlanRule{768, 512, 2, 4, 1024, 2, 2} : PlanRule{512, 512, 4, 16, 480, 2, 2});
  return plan_planes(units, L_max, r, most_split, heads_one_by_one(group), [&](int parts) {
    return column_tiles(planes_tile_rows(dtype, head_dim, parts, heads_one_by_one(group) > 1), group, L_max);
  });
}

// The schedule of one or two shares: the wide kernels' pairs for bf16 / 128; else pairs of blocks of 128 rows, with 64 rows
// (where the waves can share them) and / or two shares where `target` workgroups are not reached, and single blocks where even
// that leaves compute units idle.
inline PassPlan plan_of_two_shares(int dtype, int head_dim, long long streams, int units, int L_max, bool may_split) {
  if (dtype == 1 && head_dim == 128) {
    const int ids = ceil_div(ceil_div(L_max, 256), 2);
    return {true, 1, may_split && static_cast<long long>(units) * ids < 1024 ? 2 : 1, 1, ids};
  }
  const int target = dtype == 1 ? 1024 : 512, blocks = ceil_div(L_max, 128);
  const bool may_part = dtype == 1 || head_dim == 64;
  const long long pairs = streams * ceil_div(blocks, 2);
  PassPlan p = {false, 1, 1, 1, 0};
  if (pairs < target) {
    const bool both = 2 * pairs < target;
    if (may_part && (dtype == 1 || both || !may_split)) p.parts = 2;
    if (may_split && (dtype == 0 || both) && blocks > 1) p.split = 2;
  }
  const int own = ceil_div(L_max, 128 / p.parts);
  p.paired = streams * ceil_div(own, 2) * p.split >= 256 ? 1 : 0;
  p.ids = p.paired ? ceil_div(own, 2) : own;
  return p;
}

// What a pass's workgroups cost, in the time that a compute unit full of them takes for a tile of each of its workgroups.  Fitted
// to 800 prompts with every schedule timed (1 to 1000 units, 1 to 9 heads, 134 to 7300 tokens, ragged and not).
struct PassCost {
  int resident;               // workgroups that a compute unit holds
  float tile[3], wide;        // a streamed tile with 1, 2, 4 parts; of the wide kernels
  float own, own_wide;        // what comes with a block of owned rows: the rows, the first tiles, the sums
  float alone;                // how much longer than its share of a full compute unit's time a workgroup takes by itself
  float tail = 1.25f;         // longest blocks that the end of more single blocks than run at a time lasts
};

// Time of the pass if its workgroups are `share` of those of the plan.  tiles: streamed tiles of the longest block.
inline float estimate(const PassCost& c, const PassPlan& p, long long streams, int L_max, int tiles, float share) {
  constexpr float kUnits = 256.0f;  // compute units
  const int blocks = ceil_div(L_max, p.wide ? 256 : 128 / p.parts);
  const float n = share * static_cast<float>(streams) * static_cast<float>(p.ids) * static_cast<float>(p.split);
  const float resident = static_cast<float>(p.wide ? 2 : c.resident), own = p.wide ? c.own_wide : c.own;
  const float walk = (p.wide ? c.wide : c.tile[p.parts >> 1]) * static_cast<float>(tiles) / static_cast<float>(p.split);
  const float mean = walk * static_cast<float>(blocks + 1) / static_cast<float>(2 * blocks) + own, longest = walk + own;
  if (p.paired) {  // all alike: rounds, of which the last may leave compute units with fewer workgroups, or without
    const float full = floorf(n / (kUnits * resident)), left = ceilf(n / kUnits - full * resident);
    return (blocks == 1 ? longest : 2.0f * mean) * (full * resident + (left <= 0.0f ? 0.0f : left < c.alone ? c.alone : left));
  }
  // The longest first: where all run at a time some compute unit has the longest of every rank, else short ones fill the end.
  if (n > kUnits * resident) return mean * n / kUnits + (p.split == 1 ? c.tail : 1.25f) * longest;
  const float ranks = mean * n / kUnits + 2.0f * (longest - mean);
  return ranks > c.alone * longest ? ranks : c.alone * longest;
}

// `filling`, unless the schedule of two shares is estimated to take 6 % less, or anything less where both are the wide kernels'
// pairs, whose times the estimate does not have to compare with those of other kernels.  (Three quarters of the workgroups:
// prompts of different lengths, which the host does not know.)  tiles(plan): streamed tiles of the longest block.
template <class TilesFn>
inline PassPlan quicker_plan(const PassPlan& filling, const PassPlan& two, const PassCost& filling_cost, const PassCost& two_cost,
                             long long streams, int L_max, int most_split, TilesFn tiles) {
  if (two.split > most_split) return filling;
  const auto time = [&](const PassCost& c, const PassPlan& p) {
    return estimate(c, p, streams, L_max, tiles(p), 1.0f) + 0.5f * estimate(c, p, streams, L_max, tiles(p), 0.75f);
  };
  return time(two_cost, two) < (filling.wide && two.wide ? 1.0f : 0.94f) * time(filling_cost, filling) ? two : filling;
}

inline PassPlan plan_rows(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
  static constexpr PassCost kCost[2][2] = {{{3, {1.0f, 0.65f, 1.0f}, 0.0f, 0.75f, 0.0f, 1.4f}, {2, {1.0f, 1.0f, 1.0f}, 0.0f, 1.5f, 0.0f, 1.8f, 1.8f}},
                                           {{4, {1.0f, 0.6f, 0.35f}, 0.0f, 0.5f, 0.0f, 1.6f}, {2, {1.0f, 0.65f, 0.6f}, 0.6f, 0.75f, 1.5f, 1.4f}}};
  const PassCost& cost = kCost[dtype][head_dim == 128];
  const long long streams = static_cast<long long>(units) * group;
  return quicker_plan(filling_rows(dtype, head_dim, units, group, L_max, most_split),
                      plan_of_two_shares(dtype, head_dim, streams, units, L_max, group == 1), cost, cost, streams, L_max, most_split,
                      [&](const PassPlan& p) { return ceil_div(L_max, p.wide ? 64 : planes_tile_rows(dtype, head_dim, p.parts, false)); });
}

inline PassPlan plan_columns(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
  static constexpr PassCost kCost[2][2] = {{{3, {1.0f, 0.65f, 1.0f}, 0.0f, 1.0f, 0.0f, 2.4f}, {2, {1.0f, 1.8f, 1.0f}, 0.0f, 2.0f, 0.0f, 1.8f, 1.8f}},
                                           {{4, {1.0f, 0.55f, 0.5f}, 0.0f, 1.0f, 0.0f, 2.4f}, {2, {1.0f, 0.65f, 0.8f}, 0.6f, 0.75f, 1.5f, 1.4f}}};
  const PassPlan filling = filling_columns(dtype, head_dim, units, group, L_max, most_split);
  PassCost cost = kCost[dtype][head_dim == 128];
  const int heads = heads_one_by_one(group);
  if (heads > 1) {
    // (the wide kernel has no pipelined form for such groups: 64 units x 15 heads x 1000 tokens 735 us against 535)
    if (dtype == 1 && head_dim == 128) return filling;
    cost.own *= static_cast<float>(heads);
    if (dtype == 1) cost.tile[0] = 1.15f;  // (spills 40 registers)
  }
  PassCost alone = cost;
  if (dtype == 0 && head_dim == 128 && filling.parts == 2) alone.resident = 1;  // (tiles of 64 rows fill the LDS)
  return quicker_plan(filling, plan_of_two_shares(dtype, head_dim, units, units, L_max, true), alone, cost, units, L_max, most_split,
                      [&](const PassPlan& p) {
                        const bool small = heads_one_by_one(group) > 1;
                        return column_tiles(p.wide ? 64 : planes_tile_rows(dtype, head_dim, p.parts, small), group, L_max);
                      });
}

// Whether the column pass merges the normalisers of a row pass that several workgroups divided, as it stages them: the kernels
// of prefill_planes.hip do, if the workspace has planes for them that the pass does not write.  A launch less, 5 us of a call
// (96 x <= 1000 tokens of fp32 / 64 103.2 -> 100.6).
inline bool columns_merge_normalisers(PrefillArgs& a, const PassPlan& rows, const PassPlan& columns) {
  if (rows.split == 1 || columns.wide || a.pol.keeps_last_score()) return false;
  const size_t need = static_cast<size_t>(rows.split - 1) * a.units * a.group * a.L_max;
  if (columns.split > a.shares || need > 2 * static_cast<size_t>(a.shares - columns.split) * a.plane) return false;
  a.lse_shares = rows.split;
  a.lse_behind = 2 * columns.split;
  return true;
}

// Pairs of column sums (PrefillArgs::sums_of) that a call makes use of if its workspace has them, planes for the normalisers
// above among them; two are always there.
inline int prefill_query_shares(int dtype, int head_dim, int units, int group, int L_max) {
  const PassPlan columns = plan_columns(dtype, head_dim, units, group, L_max, kMaxQueryShares);
  int shares = columns.split;
  if (!columns.wide) shares += ceil_div((plan_rows(dtype, head_dim, units, group, L_max, kMaxKeyShares).split - 1) * group, 2);
  return shares > 2 ? shares : 2;
}

}  // namespace roco
