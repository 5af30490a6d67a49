// Pieces shared by the matrix-core prefill passes: the mapping of workgroups to units, and what a lane does with the 16
// scores of a 32x32 tile (row pass: online log-sum-exp; column pass: sums of probabilities).
#pragma once
#include "mfma.hpp"
#include "stream.hpp"

namespace roco {
namespace mfma {

// Workgroup -> (unit, block-pair) mapping.  The hardware hands consecutive workgroup ids to the 8 accelerator
// dies in turn and each die has its own L2, so the workgroups of one unit (which all stream the same K or Q
// tiles, at about the same time) are given ids that are congruent modulo 8: they land on one die and all but
// the first fetch of a tile hit its L2.  That holds for the units that fill all dies evenly, units / 8 * 8 of them.  Whole units
// would leave dies without work if the few units left over were treated so: those share the dies out evenly, four
// units two dies each, two or six units four dies each, any other number all dies for every unit (whole units on whole dies: 2
// units x 8 heads x 4396 tokens of bf16 / 64 with output took 640 us, 3 x 8 x 2578 of fp32 / 64 679; now 363 and 458).  Seven,
// or six behind others, leave so few dies without work that a unit's own L2 is worth more, if the unit more that a die then has
// does not make for one more round of workgroups (38 x 6597 tokens of bf16 / 128: 65 workgroups on dies that hold 64, 480 us
// against 604) and all dies are done within three rounds.  260 prompts of 7 to 126 units in all forms, shared against whole
// dies, geometric means: one round 1.03, two 1.03, three 1.02, more 0.99; six units by themselves and five left over 0.99 to
// 1.01, fewer (9, 12, 20, 25, 28, 36, 100 units) 0.94 to 0.99.  The grid is one-dimensional over workgroup_ids(units, whole,
// pairs) ids.
// whole: the units that go to whole dies, a multiple of 8 (up to two more than there are); resident: workgroups that a compute
// unit holds.
inline int units_on_whole_dies(int units, int pairs, int resident) {
  const int even = units & ~7;
  if (units < 7 || units - even < 6) return even;
  const long long holds = 32ll * resident, more = static_cast<long long>(even / 8 + 1) * pairs;
  const long long shared = (static_cast<long long>(units) * pairs + 7) / 8, rounds = (more + holds - 1) / holds;
  return rounds <= 3 && rounds == (shared + holds - 1) / holds ? even + 8 : even;
}
inline unsigned workgroup_ids(int units, int whole, int pairs) {
  const unsigned rest = units > whole ? static_cast<unsigned>(units - whole) : 0u;
  return static_cast<unsigned>(whole) * pairs + (rest * pairs + 7) / 8 * 8;
}
__device__ __forceinline__ bool locate(int units, int whole, int pairs, int& unit, int& pair) {
  const int lin = blockIdx.x, seq = lin >> 3;
  if (seq * 8 < whole * pairs) {
    unit = (seq / pairs) * 8 + (lin & 7);
    pair = seq % pairs;
    return unit < units;
  }
  const int rest = units & 7, groups = rest & -rest;  // of units and of dies: 1, 2 or 4
  const int die = lin & 7, per = 8 / groups;          // dies of a group
  const int k = (seq - (whole >> 3) * pairs) * per + die / groups;  // among the workgroups of the die's group of units
  unit = whole + die % groups + groups * (k / pairs);
  pair = k % pairs;
  return unit < units;
}
// The same for (unit, query head) pairs, u = unit * group + head: the heads of a unit stream the same keys (and
// values), so they share a die, one head after the other.  The grid covers workgroup_ids(units, whole, group * pairs)
// ids.
__device__ __forceinline__ bool locate_heads(int units, int whole, int group, int pairs, int& u, int& pair) {
  int unit, id;
  if (!locate(units, whole, group * pairs, unit, id)) return false;
  u = unit * group + id / pairs;
  pair = id % pairs;
  return true;
}

// Online log-sum-exp update of one lane with the 16 scores of a tile.
//   INTERIOR: every key of the tile is visible to every query of the group and none is inside a recency window:
//             3 vector instructions per score (multiply-add, exponential, add) plus 8 for the maximum.
// l = sum 2^(t - m) is a floating-point number, so m need not be the running maximum: any reference that keeps the
// terms from overflowing gives the same sum to rounding.  The terms of a tile are first taken against the reference
// as it stands (3 instructions per score and nothing else: `sum`); only if some lane's share comes out above 2^64
// -- the first tile, whose reference is -inf, and a row whose scores later rise by more than 64 powers of two --
// is the tile redone with the reference raised to its maximum.
__device__ __forceinline__ void lazy_finish(float sum, const f32x16& s, float sc, float& m, float& l) {
  if (__builtin_amdgcn_ballot_w64(!(sum <= 0x1p64f)) == 0) {
    l += sum;
  } else {
    const float m_new = fmaxf(m, max16(s) * sc);
    if (m_new > -INFINITY) {  // false while every logit of the lane has been -inf: those terms are zero
      const float neg_new = -m_new;
      float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        t0 += fast_exp2(fmaf(s[r], sc, neg_new));
        t1 += fast_exp2(fmaf(s[r + 1], sc, neg_new));
      }
      l = fmaf(l, fast_exp2(m - m_new), t0 + t1);
      m = m_new;
    }
  }
}

template <bool INTERIOR>
__device__ __forceinline__ void lse_update(const f32x16& s, float sc, int kb, int half, int qi, int w, float rb,
                                           float& m, float& l) {
  if (INTERIOR) {
    const float neg = -m;
    float sum0 = 0.0f, sum1 = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      sum0 += fast_exp2(fmaf(s[r], sc, neg));
      sum1 += fast_exp2(fmaf(s[r + 1], sc, neg));
    }
    lazy_finish(sum0 + sum1, s, sc, m, l);
  } else {
    float tv[16];
    float mb = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = kb + 8 * (r >> 2) + 4 * half + (r & 3);
      float x = s[r] * sc;
      if (w > 0 && qi - key < w) x += rb;
      if (key > qi) x = -INFINITY;
      tv[r] = x;
      mb = fmaxf(mb, x);
    }
    const float m_new = fmaxf(m, mb);
    if (m_new > -INFINITY) {
      float sum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += fast_exp2(tv[r] - m_new);
      l = l * fast_exp2(m - m_new) + sum;
      m = m_new;
    }
  }
}

// Column-statistics update of one lane (one key) with the 16 scores of a tile (16 queries).  COUNT: the second
// statistic is the number of queries that gave the key more than their row's average, p * (i + 1) > 1 (section
// 4.1, quantised score), instead of the sum of squares.
template <bool INTERIOR, bool COUNT>
__device__ __forceinline__ void column_update(const f32x16& s, const float* lse_tile, const float* rinv_tile, float sc,
                                              int ib, int half, int kj, int len, int w, float rb, float& s1, float& s2) {
  float a1 = 0.0f, a2 = 0.0f, b1 = 0.0f, b2 = 0.0f;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const float4 ls = *reinterpret_cast<const float4*>(lse_tile + 8 * g4 + 4 * half);
    const float lv[4] = {ls.x, ls.y, ls.z, ls.w};
    float rv[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // COUNT: 1 / (tokens the query attended), staged with the normalisers
    if (COUNT) {
      const float4 rs = *reinterpret_cast<const float4*>(rinv_tile + 8 * g4 + 4 * half);
      rv[0] = rs.x; rv[1] = rs.y; rv[2] = rs.z; rv[3] = rs.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = fmaf(s[4 * g4 + e], sc, -lv[e]);
      float p;
      if (INTERIOR) {
        p = fast_exp2(x);
      } else {
        const int qi = ib + 8 * g4 + 4 * half + e;
        if (w > 0 && qi - kj < w) x += rb;
        p = fast_exp2(x);
        if (qi < kj || qi >= len) p = 0.0f;
      }
      float second;
      if (COUNT) {
        second = p > rv[e] ? 1.0f : 0.0f;  // p * (i + 1) > 1
      } else {
        second = p * p;
      }
      if (e & 1) { b1 += p; b2 = COUNT ? b2 + second : fmaf(p, p, b2); }
      else       { a1 += p; a2 = COUNT ? a2 + second : fmaf(p, p, a2); }
    }
  }
  s1 += a1 + b1;
  s2 += a2 + b2;
}

// The 16 probabilities of a tile (one key, 16 queries of one head) added into `pb` (cleared before the first head).
template <bool INTERIOR>
__device__ __forceinline__ void column_probs(const f32x16& s, const float* lse_tile, float sc, int ib, int half,
                                             int kj, int len, int w, float rb, f32x16& pb) {
  if (!INTERIOR) {
    // The masks of this (rare) path depend only on values known before the branch that leads here; the compiler
    // would compute all of them ahead of that branch, on every tile.  An opaque copy of the block index keeps them here.
    asm volatile("" : "+s"(ib));
  }
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const float4 ls = *reinterpret_cast<const float4*>(lse_tile + 8 * g4 + 4 * half);
    const float lv[4] = {ls.x, ls.y, ls.z, ls.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = fmaf(s[4 * g4 + e], sc, -lv[e]);
      float p;
      if (INTERIOR) {
        p = fast_exp2(x);
      } else {
        const int qi = ib + 8 * g4 + 4 * half + e;
        if (w > 0 && qi - kj < w) x += rb;
        p = fast_exp2(x);
        if (qi < kj || qi >= len) p = 0.0f;
      }
      pb[4 * g4 + e] += p;
    }
  }
}

// Row order of a streamed tile that holds 2 (16 / G) query positions per 32 rows for all G heads of a group, G <= 16: the
// heads of a query land in G consecutive accumulator registers of a lane (register r of lane half hf holds row
// 8 * (r / 4) + 4 * hf + r % 4 of a 32-row sub-tile; that row is given to query hf * (16 / G) + r / G of the sub-tile, head
// r % G), so the sum over the heads is a sum down a few registers of one result tile.  Where G does not divide 16 the last
// 16 % G registers of a lane repeat the row before them and are not looked at.
template <int G> struct GroupedRows {
  static constexpr int kPerHalf = 16 / G;         // queries per lane half in a 32-row sub-tile
  static constexpr int kUsed = kPerHalf * G;      // registers of a lane that hold a score
  static constexpr int kPerSub = 2 * kPerHalf;    // query positions per sub-tile
  static constexpr int kPerTile = 2 * kPerSub;    // query positions per 64-row tile
  // LDS row of a tile -> local query position and head
  __device__ static void locate(int row, int& ql, int& h) {
    const int sub = row >> 5, rr = row & 31;
    const int hf = (rr >> 2) & 1, reg = 4 * (rr >> 3) + (rr & 3), r = reg < kUsed ? reg : kUsed - 1;
    ql = sub * kPerSub + hf * kPerHalf + r / G;
    h = r % G;
  }
};

template <bool INTERIOR, int G>
__device__ __forceinline__ void column_update_grouped(const f32x16& s, const float* lse_tile, float sc, int ib, int half,
                                                      int kj, int len, int w, float rb, const Policy& pol,
                                                      float& s1, float& s2) {
  if (!INTERIOR) asm volatile("" : "+s"(ib));  // keeps this path's masks out of the code before the branch (see column_probs)
  constexpr int kPerHalf = GroupedRows<G>::kPerHalf;
  float p[16];
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const float4 ls = *reinterpret_cast<const float4*>(lse_tile + 8 * g4 + 4 * half);
    const float lv[4] = {ls.x, ls.y, ls.z, ls.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * g4 + e;
      if (r >= GroupedRows<G>::kUsed) continue;
      float x = fmaf(s[r], sc, -lv[e]);
      if (INTERIOR) {
        p[r] = fast_exp2(x);
      } else {
        const int qi = ib + half * kPerHalf + r / G;
        if (w > 0 && qi - kj < w) x += rb;
        p[r] = (qi < kj || qi >= len) ? 0.0f : fast_exp2(x);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kPerHalf; ++q) {
    float sum = p[q * G];
#pragma unroll
    for (int h = 1; h < G; ++h) sum += p[q * G + h];
    const float pbar = sum * (1.0f / static_cast<float>(G));
    s1 += pbar;
    s2 = pol.second_statistic(s2, pbar, static_cast<float>(ib + half * kPerHalf + q + 1));
  }
}

}  // namespace mfma
// The base-2 log-sum-exp of a row from those of its `shares` shares of keys (the first, and the others in `more`).
__device__ __forceinline__ float merged_normaliser(float first, const float* more, int shares) {
  float top = first;
#pragma unroll
  for (int k = 1; k < kMaxKeyShares; ++k) top = k < shares ? fmaxf(top, more[k - 1]) : top;
  if (!(top > -INFINITY)) return first;
  float sum = fast_exp2(first - top);
#pragma unroll
  for (int k = 1; k < kMaxKeyShares; ++k) sum += k < shares ? fast_exp2(more[k - 1] - top) : 0.0f;
  return top + log2f(sum);
}

}  // namespace roco
