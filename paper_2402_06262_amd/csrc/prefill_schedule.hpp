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
// The constants are those of least regret over 310 prompts with every schedule timed (1 to 1024 units, 1 to 8 heads, 100 to
// 16384 tokens, ragged and not): what they pick takes 5 % longer than the best schedule.  Column pass, us, with two shares and
// 64 owned rows at most -> now:
//   1 unit  x 8 heads x 3852 tokens of fp32 / 128  823 -> 125     2 units x 8 x 4396 of bf16 / 64   178 -> 60
//   3 units x 8 heads x 515 tokens of bf16 / 128    73 -> 12      1 unit  x 4 x 426 of bf16 / 128    30 -> 8
#pragma once
#include "kernels.hpp"

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

template <class TilesFn>
inline PassPlan plan_planes(long long streams, int L_max, const PlanRule& r, int most_split, TilesFn tiles) {
  PassPlan p = {false, 1, 1, 1, ceil_div(ceil_div(L_max, 128), 2)};
  const long long pairs = streams * p.ids;
  p.split = r.resident != 0 ? rounds_split(pairs, r.resident, tiles(1), 6.0, most_split) : power_of_two_from(r.paired_want, pairs);
  if (p.split <= most_split && p.split <= r.paired_split && pairs * p.split >= r.paired_want && tiles(1) >= r.paired_tiles * p.split) return p;
  long long best = 0;
  for (int parts = 1; parts <= r.most_parts; parts *= 2) {
    const int ids = ceil_div(L_max, 128 / parts);
    int split = power_of_two_from(r.single_want, streams * ids);
    while (split > 1 && (split > most_split || tiles(parts) < r.single_tiles * split)) split /= 2;
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
inline PassPlan plan_rows(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
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
  return plan_planes(streams, L_max, r, most_split,
                     [&](int parts) { return ceil_div(L_max, planes_tile_rows(dtype, head_dim, parts, false)); });
}

inline PassPlan plan_columns(int dtype, int head_dim, int units, int group, int L_max, int most_split) {
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
  return plan_planes(units, L_max, r, most_split, [&](int parts) {
    return column_tiles(planes_tile_rows(dtype, head_dim, parts, group > 1 && !heads_in_tile(group)), group, L_max);
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
