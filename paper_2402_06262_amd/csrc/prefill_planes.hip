// Prefill attention statistics on the gfx950 matrix cores for fp32 storage and for head_dim 64.
//
// The two passes of prefill_mfma.hip (row normalisers, column statistics) and the same orientation: a workgroup of four
// waves owns 32 or 64 rows of one operand per wave, in registers, as B operands of v_mfma_f32_32x32x16_bf16; the other
// operand streams past them through LDS; in the 32x32 result tile the owned row is the lane and the streamed rows run
// down the 16 accumulator registers, so the reductions of a pass cross no lanes.
//
// fp32 operands are taken apart into three bf16 planes, x = hi + mid + lo, each the round-to-nearest bf16 of what the
// planes before it left over: 24 significand bits in all, the width of fp32.  A product keeps the six terms of 2^-16 and
// above (hi hi, hi mid, mid hi, hi lo, lo hi, mid mid; every one is exact in fp32) and drops those of 2^-24.  The five
// small terms run on accumulator chains of their own and are added to the hi-hi sum once per tile, so a logit sees one
// rounding per 16 products at its own magnitude.  Six bf16 instructions cover 16 k-elements in 192 matrix cycles; the
// fp32 instruction (32x32x2) needs 512.
//
// What bounds the passes (counters, 128 streams x 2048 tokens of bf16 / 64, four heads): a 32x32 tile takes 81 vector
// instructions in the row pass and 98 in the column pass, 392 and 457 issue cycles where multiply-adds, exponentials and
// additions alone need 256 and 320, against 128 matrix cycles.  The vector ALUs are busy 77 and 72 % of the time, the matrix
// pipe 25 and 20 %, half of that beside a vector instruction, neither of them 11 and 18 %: vector issue above all, and what
// one wave's chain of scores, exponentials and sums leaves idle although two to four workgroups per compute unit overlap.
// fp32 / 64 (96 ragged units of up to 1000 tokens): vector ALUs 56 and 55 %, matrix pipe 38 and 34 %, neither 20 and 23 %:
// exponentials and operand splitting, then products, and the start and end of short streams.  Nothing is pipelined by hand.
//
// What three planes do not hold exactly -- infinities and NaN, values from 2^127 on, which may round to infinity, nonzero
// values below 2^-110, whose last bits are below bf16's range -- stays off the matrix cores: a wave that owns such a row, and
// every wave for a streamed tile that holds one, multiplies the fp32 numbers themselves on the vector ALUs.  So does the
// product with such values of V, and with infinite bf16 ones, which may reach only the queries that see their key.  (32 units
// x 2048 tokens of nothing but such values: 2.3 ms without and 3.4 with output for fp32 / 64, 3.8 and 11.6 for fp32 / 128,
// where the passes of prefill_simple.hip take 2.1 and 4.2.  Probabilities below 2^-110 of their row's reference keep an error
// of 2^-134 of it.)  A tile with values of V from 2^65 on goes the same way, with its row's true maximum as the reference:
// against a lazily raised one the unnormalised output may be 2^16 times larger, and overflow where the output does not.
#include "kernels.hpp"
#include "mfma.hpp"
#include "prefill_schedule.hpp"
#include "prefill_tiles.hpp"
#include "profile.hpp"
#include "stream.hpp"

namespace roco {
namespace {

using mfma::bf16x8;
using mfma::f32x16;
using mfma::column_probs;
using mfma::column_update;
using mfma::column_update_grouped;
using mfma::GroupedRows;
using mfma::lds_read_transposed;
using mfma::locate;
using mfma::locate_heads;
using mfma::lse_update;
using mfma::max16;

constexpr int kThreads = 256;

// Rows of a streamed tile: as many as leave room for the resident workgroups (bf16: 128, fewer barriers per row; the kernels
// with an output tile or head sums next to their scores take 64).
template <int DT, int D> constexpr int kRows = DT == kBF16 ? 128 : D == 128 ? 32 : 64;
template <int DT, int D> constexpr int kRowsSmall = DT == kF32 && D == 128 ? 32 : 64;

// Geometry of a streamed tile: TR rows of NP bf16 planes in LDS.
template <int DT, int D, int ROWS> struct Planes {
  static constexpr int NP = DT == kF32 ? 3 : 1;
  static constexpr int KS = D / 16;                         // k-steps of the 32x32x16 instruction
  static constexpr int TR = ROWS;
  static constexpr int SUBS = TR / 32;
  static constexpr int ROW = 2 * D;                         // bytes of a plane row
  static constexpr int PLANE = TR * ROW;
  static constexpr int TILE = NP * PLANE;
  // V rows: a 16-lane group of a transpose read touches 4 rows x 32 bytes, which then lie on distinct banks
  static constexpr int ROWV = ROW + 64;
  static constexpr int PLANEV = TR * ROWV;
  static constexpr int TILEV = NP * PLANEV;
  static constexpr int IN_ROW = D * (DT == kF32 ? 4 : 2);   // bytes of a row in memory
  static constexpr int CPR = IN_ROW / 16;                   // 16-byte chunks per row
  static constexpr int PIECES = TR * CPR / kThreads;        // chunks per thread and tile
  static_assert(TR * CPR % kThreads == 0, "a tile is dealt evenly to the threads");
};

// 16-byte chunk `ch` of plane row `row`: stored in a slot that makes the 128-bit fragment reads (16 consecutive rows, same
// chunk) fall on 16 distinct groups of banks.  Rows of 128 bytes share the banks of two rows, hence the shift.
template <int D> __device__ __forceinline__ int chunk_offset(int row, int ch) {
  return row * 2 * D + ((D == 64 ? ch ^ ((row >> 1) & 7) : ch ^ (row & 15)) << 4);
}

// Four fp32 values as three planes of four bf16 values, exact for zeros and for values in [2^-110, 2^127).
__device__ __forceinline__ void split4(const uint4& w, uint2* p) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto pack = [](f32x2 v) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)); };
  auto less = [](f32x2 v, uint32_t h) {  // what a plane leaves over: exact
    return f32x2{v.x - __uint_as_float(h << 16), v.y - __uint_as_float(h & 0xffff0000u)};
  };
  f32x2 a = {__uint_as_float(w.x), __uint_as_float(w.y)}, b = {__uint_as_float(w.z), __uint_as_float(w.w)};
  p[0] = make_uint2(pack(a), pack(b));
  a = less(a, p[0].x);
  b = less(b, p[0].y);
  p[1] = make_uint2(pack(a), pack(b));
  a = less(a, p[1].x);
  b = less(b, p[1].y);
  p[2] = make_uint2(pack(a), pack(b));
}
// Whether values lie outside that range.  An offset from its lower end that wraps around for anything smaller, one maximum
// over all of a thread's values and one comparison; only if that fails (zeros wrap around too) are they looked at one by one.
constexpr uint32_t kPlanesFrom = 17u << 24, kPlanesTo = 254u << 24;  // twice the bits of 2^-110 and 2^127: no sign
constexpr uint32_t kValuesTo = 192u << 24;                          // ... and of 2^65 (see the head of the file)
__device__ __forceinline__ uint32_t planes_offset(uint32_t bits) { return (bits << 1) - kPlanesFrom; }
__device__ __forceinline__ uint32_t farthest(uint32_t far, const uint4& w) {
  far = max(max(far, planes_offset(w.x)), planes_offset(w.y));
  return max(max(far, planes_offset(w.z)), planes_offset(w.w));
}
template <uint32_t TO, int N> __device__ __forceinline__ bool outside_planes(uint32_t far, const uint4 (&w)[N]) {
  if (__builtin_expect(far < TO - kPlanesFrom, 1)) return false;
  bool odd = false;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t u[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) odd |= (u[e] << 1) != 0u && planes_offset(u[e]) >= TO - kPlanesFrom;
  }
  return odd;
}
__device__ __forceinline__ f32x16 mm(const uint4& x, const uint4& y, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
}

// A thread's chunks of a tile on their way from memory to LDS.
template <int DT, int D, int ROWS> struct Pieces {
  using P = Planes<DT, D, ROWS>;
  uint4 w[P::PIECES];
  __device__ __forceinline__ void load(const char* base, int row0, int last_row) {
#pragma unroll
    for (int i = 0; i < P::PIECES; ++i) {
      const int idx = threadIdx.x + kThreads * i;
      const int row = min(row0 + idx / P::CPR, last_row);  // rows past the end are masked by the caller
      w[i] = load16(base + static_cast<size_t>(row) * P::IN_ROW + (idx % P::CPR) * 16);
    }
  }
  // Rows of a tile that holds the query positions from `pos0` on for G heads (see GroupedRows), head h at base + h * stride.
  template <int G> __device__ __forceinline__ void load_heads(const char* base, size_t stride, int pos0, int last_pos) {
#pragma unroll
    for (int i = 0; i < P::PIECES; ++i) {
      const int idx = threadIdx.x + kThreads * i;
      int ql, h;
      GroupedRows<G>::locate(idx / P::CPR, ql, h);
      const int pos = min(pos0 + ql, last_pos);
      w[i] = load16(base + h * stride + static_cast<size_t>(pos) * P::IN_ROW + (idx % P::CPR) * 16);
    }
  }
  // Into the planes of a K or Q tile; true if this thread met a value they do not hold (fp32 only).
  __device__ __forceinline__ bool store(char* tile) const {
    uint32_t far = 0;
#pragma unroll
    for (int i = 0; i < P::PIECES; ++i) {
      const int idx = threadIdx.x + kThreads * i;
      const int row = idx / P::CPR, c = idx % P::CPR;
      if constexpr (DT == kBF16) {
        *reinterpret_cast<uint4*>(tile + chunk_offset<D>(row, c)) = w[i];
      } else {
        uint2 p[3];
        split4(w[i], p);
        far = farthest(far, w[i]);
        char* at = tile + chunk_offset<D>(row, c >> 1) + (c & 1) * 8;
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(at + k * P::PLANE) = p[k];
      }
    }
    return DT == kF32 && outside_planes<kPlanesTo>(far, w);
  }
  // Into the planes of a V tile (rows of ROWV bytes); true if this thread met a value they do not hold or one from 2^65 on.
  __device__ __forceinline__ bool store_values(char* tile) const {
    uint32_t far = 0, large = 0;
#pragma unroll
    for (int i = 0; i < P::PIECES; ++i) {
      const int idx = threadIdx.x + kThreads * i;
      const int row = idx / P::CPR, c = idx % P::CPR;
      if constexpr (DT == kBF16) {
        // the two upper bits of the exponent fields: set from 2^65 on
        large |= (w[i].x & (w[i].x << 1)) | (w[i].y & (w[i].y << 1)) | (w[i].z & (w[i].z << 1)) | (w[i].w & (w[i].w << 1));
        *reinterpret_cast<uint4*>(tile + row * P::ROWV + c * 16) = w[i];
      } else {
        uint2 p[3];
        split4(w[i], p);
        far = farthest(far, w[i]);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(tile + k * P::PLANEV + row * P::ROWV + c * 8) = p[k];
      }
    }
    if constexpr (DT == kBF16) return (large & 0x40004000u) != 0u;
    return outside_planes<kValuesTo>(far, w);
  }
};

// This lane's row of one group of 32 owned rows, as B operands.
template <int DT, int D> struct Owned {
  using P = Planes<DT, D, 64>;
  uint4 f[P::NP][P::KS];
  // true if the lane met a value that the planes do not hold
  __device__ __forceinline__ bool load(const char* base, int row, int last_row) {
    const int half = (threadIdx.x & (kWave - 1)) >> 5;
    const char* at = base + static_cast<size_t>(min(row, last_row)) * P::IN_ROW;
    if constexpr (DT == kBF16) {
#pragma unroll
      for (int kk = 0; kk < P::KS; ++kk) f[0][kk] = load16(at + kk * 32 + half * 16);
      return false;
    } else {
      uint32_t far = 0;
      uint4 w[2 * P::KS];
#pragma unroll
      for (int kk = 0; kk < P::KS; ++kk) {
        uint2 a[3], b[3];
        w[2 * kk] = load16(at + kk * 64 + half * 32);
        w[2 * kk + 1] = load16(at + kk * 64 + half * 32 + 16);
        far = farthest(farthest(far, w[2 * kk]), w[2 * kk + 1]);
        split4(w[2 * kk], a);
        split4(w[2 * kk + 1], b);
#pragma unroll
        for (int k = 0; k < 3; ++k) f[k][kk] = make_uint4(a[k].x, a[k].y, b[k].x, b[k].y);
      }
      return outside_planes<kPlanesTo>(far, w);
    }
  }
};

// Score tile: the 32 streamed rows of sub-tile `sub` against 32 owned rows.
template <int ROWS, int DT, int D>
__device__ __forceinline__ f32x16 score_tile(const char* tile, int sub, const Owned<DT, D>& own) {
  using P = Planes<DT, D, ROWS>;
  const int lane = threadIdx.x & (kWave - 1);
  const int row = sub * 32 + (lane & 31);
  const f32x16 zero = {0};
  f32x16 acc;
  auto frag = [&](int plane, int kk) {
    return *reinterpret_cast<const uint4*>(tile + plane * P::PLANE + chunk_offset<D>(row, 2 * kk + (lane >> 5)));
  };
  if constexpr (DT == kBF16) {
#pragma unroll
    for (int kk = 0; kk < P::KS; ++kk) acc = mm(frag(0, kk), own.f[0][kk], kk == 0 ? zero : acc);
  } else {
    // The small terms share one chain: a second one would let a wave issue them back to back, but the registers it takes
    // are worth more as a third resident wave (fp32 / 64, 64 units x 2048 tokens: 112 us per pass against 137).
    f32x16 small = zero;
#pragma unroll
    for (int kk = 0; kk < P::KS; ++kk) {
      const uint4 h = frag(0, kk), m = frag(1, kk), l = frag(2, kk);
      small = mm(l, own.f[0][kk], small);
      small = mm(h, own.f[2][kk], small);
      acc = mm(h, own.f[0][kk], kk == 0 ? zero : acc);
      small = mm(m, own.f[1][kk], small);
      small = mm(h, own.f[1][kk], small);
      small = mm(m, own.f[0][kk], small);
    }
    acc += small;
  }
  return acc;
}
// The same tile from the fp32 rows themselves: `row_at(i)` is the address of streamed row i of the sub-tile, `own_row` of the
// lane's owned row.  Four streamed rows at a time, which keeps the registers of this rare path out of the kernel's way.
template <int D, class RowAt>
__device__ __forceinline__ f32x16 score_tile_plain(RowAt row_at, const char* own_row) {
  const int half = (threadIdx.x & (kWave - 1)) >> 5;
  f32x16 acc = {0};
#pragma unroll 1
  for (int g4 = 0; g4 < 4; ++g4) {
    const char* at[4];
    float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) at[e] = row_at(8 * g4 + 4 * half + e);
#pragma unroll 1
    for (int c = 0; c < D * 4; c += 16) {
      float x[4];
      unpack16<kF32>(load16(own_row + c), x);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float y[4];
        unpack16<kF32>(load16(at[e] + c), y);
#pragma unroll
        for (int k = 0; k < 4; ++k) dot[e] = fmaf(x[k], y[k], dot[e]);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = (r >> 2) == g4 ? dot[r & 3] : acc[r];
  }
  return acc;
}

// Blocks of owned rows of a workgroup: paired, it takes the p-th longest and the p-th shortest (equal work whatever the
// position under the causal diagonal), else one.  Returns false when there is none for this id and pass.
__device__ __forceinline__ bool pick_block(bool paired, int pass, int pair_id, int n_blocks, bool long_last, int& blk) {
  if (!paired) {
    if (pass == 1 || pair_id >= n_blocks) return false;
    blk = long_last ? n_blocks - 1 - pair_id : pair_id;  // the longest streams start first
    return true;
  }
  const int far = n_blocks - 1 - pair_id;
  if (far < pair_id || (pass == 1 && far == pair_id)) return false;
  blk = (pass == 0) == long_last ? far : pair_id;
  return true;
}

// The four waves of a workgroup share its owned rows and the streamed tiles: PARTS = 1, every wave owns 32 rows of its own
// and takes all sub-tiles of 32 streamed rows; PARTS = 2, waves w and w + 2 own the same 32 rows and take every other
// sub-tile (twice the workgroups of half the length for the same rows); PARTS = 4, all of them own the same 32 rows and take
// one sub-tile in four.  Their results meet in LDS at the end.
template <int PARTS> struct Shares {
  static constexpr int GROUPS = 4 / PARTS;
  static constexpr int kOwn = 32 * GROUPS;
};
// Rows of a streamed tile: every part has a sub-tile of its own.
template <int DT, int D, int PARTS> constexpr int kTileRows = kRows<DT, D> > 32 * PARTS ? kRows<DT, D> : 32 * PARTS;
template <int DT, int D, int PARTS> constexpr int kTileRowsSmall = kRowsSmall<DT, D> > 32 * PARTS ? kRowsSmall<DT, D> : 32 * PARTS;

// ------------------------------------------------------------------------------------------------
// pass 1: lse[i] = log2 sum_{j<=i} 2^(t_ij)
template <int DT, int D, int PARTS>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : DT == kBF16 ? 4 : 3) void prefill_rows_planes(PrefillArgs a) {
  using P = Planes<DT, D, kTileRows<DT, D, PARTS>>;
  constexpr int kOwn = Shares<PARTS>::kOwn, GROUPS = Shares<PARTS>::GROUPS;
  __shared__ __attribute__((aligned(16))) char tiles[2][P::TILE];
  __shared__ float other[2][PARTS > 1 ? PARTS - 1 : 1][PARTS > 1 ? kOwn : 1];
  __shared__ int odd_s[2];  // number of the last tile in this buffer that holds values of no exact planes (fp32)
  int u, id;
  if (!locate_heads(a.units, a.whole, a.group, a.pairs * a.ksplit, u, id)) return;
  const int seg = id % a.ksplit, pair_id = id / a.ksplit;
  float* const lse_out = a.lse_of_share(seg);  // see merge_key_shares
  const int uk = u / a.group;
  const int len = a.len[uk];
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int half = lane >> 5, grp = wave % GROUPS, part = wave / GROUPS;
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  const char* Qb = static_cast<const char*>(a.Q) + ubase * P::IN_ROW;
  const char* Kb = static_cast<const char*>(a.K) + static_cast<size_t>(uk) * a.L_max * P::IN_ROW;
  const float sc = a.scale_log2;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const int n_blocks = (len + kOwn - 1) / kOwn;
  if (threadIdx.x == 0) odd_s[0] = odd_s[1] = 0;
  int seq = 0;  // tiles so far

  for (int pass = 0; pass < 2; ++pass) {
    int blk;
    if (!pick_block(a.paired != 0, pass, pair_id, n_blocks, true, blk)) break;
    const int q0 = blk * kOwn;
    const int qg = q0 + 32 * grp, qi = qg + (lane & 31);  // first query of the wave's group, this lane's query
    const int n_tiles = (min(len, q0 + kOwn) - 1) / P::TR + 1;
    int t_lo = 0, t_hi = n_tiles - 1;  // this workgroup's share of the key tiles (possibly none)
    if (a.ksplit > 1) {
      const int per = (n_tiles + a.ksplit - 1) / a.ksplit;
      t_lo = seg * per;
      t_hi = min(t_hi, t_lo + per - 1);
    }
    Pieces<DT, D, P::TR> st;
    if (t_lo <= t_hi) st.load(Kb, t_lo * P::TR, len - 1);
    __syncthreads();  // the previous block has finished with the tiles and what goes with them; odd_s is cleared
    Owned<DT, D> own;
    const bool odd_own = __builtin_amdgcn_ballot_w64(own.load(Qb, qi, len - 1)) != 0;
    float m = -INFINITY, l = 0.0f;
    for (int t = t_lo; t <= t_hi; ++t) {
      const int buf = (t - t_lo) & 1;
      char* const tile = tiles[buf];
      ++seq;
      if (st.store(tile) && DT == kF32) odd_s[buf] = seq;
      __syncthreads();  // tile t is in LDS; everybody is done with tile t - 1, whose buffer tile t + 1 takes
      if (t + 1 <= t_hi) st.load(Kb, (t + 1) * P::TR, len - 1);
      const bool odd = DT == kF32 && (odd_own || __builtin_amdgcn_readfirstlane(odd_s[buf]) == seq);
#pragma unroll
      for (int i = 0; i < P::SUBS / PARTS; ++i) {
        const int sub = part + PARTS * i;
        const int kb = t * P::TR + sub * 32;
        if (kb > qg + 31) continue;  // wholly above the diagonal
        f32x16 s;
        if (odd) s = score_tile_plain<D>([&](int i) { return Kb + static_cast<size_t>(min(kb + i, len - 1)) * P::IN_ROW; },
                                         Qb + static_cast<size_t>(min(qi, len - 1)) * P::IN_ROW);
        else s = score_tile<P::TR>(tile, sub, own);
        if (kb + 31 + w <= qg) lse_update<true>(s, sc, kb, half, qi, w, rb, m, l);
        else lse_update<false>(s, sc, kb, half, qi, w, rb, m, l);
      }
    }
    auto join = [&](float mo, float lo) {  // sums over other keys of the same query
      const float mn = fmaxf(m, mo);
      l = (m > -INFINITY ? l * fast_exp2(m - mn) : 0.0f) + (mo > -INFINITY ? lo * fast_exp2(mo - mn) : 0.0f);
      m = mn;
    };
    const float mo = __shfl_xor(m, 32, kWave), lo = __shfl_xor(l, 32, kWave);
    join(mo, lo);
    if constexpr (PARTS > 1) {
      if (part > 0 && half == 0) { other[0][part - 1][32 * grp + lane] = m; other[1][part - 1][32 * grp + lane] = l; }
      __syncthreads();
      if (part == 0 && half == 0) {
#pragma unroll
        for (int o = 0; o < PARTS - 1; ++o) join(other[0][o][32 * grp + lane], other[1][o][32 * grp + lane]);
      }
    }
    if (part == 0 && half == 0 && qi < len) lse_out[ubase + qi] = m + log2f(l);  // -inf for a share without keys
  }
}

// ------------------------------------------------------------------------------------------------
// pass 2: Acc[j] = sum_i Pbar[i,j], Acc2[j] = sum_i Pbar[i,j]^2 (or the count of above-average queries), Pbar the mean over
// the unit's query heads.  A workgroup owns a block of keys and walks the query tiles from the end of the prompt down to
// its own keys; grouped, a tile position is taken head by head and the sum over the heads stays in the lane's registers.
// HEADS: 1, or 0 for any group (head by head), or 2 to 8 or 16 for that group with the head sum inside a result tile.
// Waves per SIMD (fp32 / 128 with two parts: two tiles take 96 KiB).
template <int DT, int D, int PARTS, int HEADS>
constexpr int kColumnWaves = DT == kF32 && D == 128 && PARTS > 1 ? 1 : D == 128 ? 2 : DT == kBF16 ? (HEADS != 0 ? 4 : 3) : HEADS != 0 ? 3 : 2;
template <int DT, int D, int PARTS, int HEADS>
__global__ __launch_bounds__(kThreads, (kColumnWaves<DT, D, PARTS, HEADS>)) void prefill_columns_planes(PrefillArgs a) {
  using P = Planes<DT, D, HEADS == 0 ? kTileRowsSmall<DT, D, PARTS> : kTileRows<DT, D, PARTS>>;
  constexpr int kOwn = Shares<PARTS>::kOwn, GROUPS = Shares<PARTS>::GROUPS, NSUB = P::SUBS / PARTS;
  constexpr int PER = HEADS > 1 ? HEADS : 1;               // heads per query position of a tile
  constexpr int QS = HEADS > 1 ? GroupedRows<PER>::kPerSub : 32;  // query positions per sub-tile
  constexpr int QT = P::SUBS * QS;                                // ... and per tile
  __shared__ __attribute__((aligned(16))) char tiles[2][P::TILE];
  __shared__ __attribute__((aligned(16))) float lse_s[2][P::TR], rinv_s[2][P::TR];  // rinv: 1 / (tokens the query attended)
  __shared__ float other[2][PARTS > 1 ? PARTS - 1 : 1][PARTS > 1 ? kOwn : 1];
  __shared__ int odd_s[2];  // see prefill_rows_planes
  int u, id;
  if (!locate(a.units, a.whole, a.pairs * a.qsplit, u, id)) return;
  const int seg = id % a.qsplit, pair_id = id / a.qsplit;
  float *const out1 = a.sums_of(seg, 0), *const out2 = a.sums_of(seg, 1);
  const int G = HEADS != 1 ? a.group : 1;
  const float inv_heads = 1.0f / static_cast<float>(G);
  const bool count = a.pol.counts_above_average();
  const int len = a.len[u];
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int half = lane >> 5, grp = wave % GROUPS, part = wave / GROUPS;
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  const char* Kb = static_cast<const char*>(a.K) + ubase * P::IN_ROW;
  const char* Qu = static_cast<const char*>(a.Q) + ubase * G * P::IN_ROW;  // [G][L_max][d]
  const float* lse_u = a.lse + ubase * G;
  const float sc = a.scale_log2;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const int n_blocks = (len + kOwn - 1) / kOwn;
  if (threadIdx.x == 0) odd_s[0] = odd_s[1] = 0;
  int seq = 0;

  for (int pass = 0; pass < 2; ++pass) {
    int blk;
    if (!pick_block(a.paired != 0, pass, pair_id, n_blocks, false, blk)) break;
    const int j0 = blk * kOwn;
    const int kg = j0 + 32 * grp, kj = kg + (lane & 31);  // first key of the wave's group, this lane's key
    int t_first = j0 / QT, t_last = (len - 1) / QT;
    if (a.qsplit > 1) {  // this workgroup's share of the query tiles (possibly none)
      const int per = (t_last - t_first + a.qsplit) / a.qsplit;
      t_first += seg * per;
      t_last = min(t_last, t_first + per - 1);
    }
    Pieces<DT, D, P::TR> st;
    float st_lse = 0.0f, st_more[kMaxKeyShares - 1];
    auto fetch = [&](int t, int h) {
      int lse_h = h, lse_q = threadIdx.x;
      if constexpr (HEADS > 1) {
        st.template load_heads<PER>(Qu, static_cast<size_t>(a.L_max) * P::IN_ROW, t * QT, len - 1);
        GroupedRows<PER>::locate(threadIdx.x, lse_q, lse_h);
      } else {
        st.load(Qu + static_cast<size_t>(h) * a.L_max * P::IN_ROW, t * QT, len - 1);
      }
      if (threadIdx.x < P::TR) {
        const size_t at = static_cast<size_t>(lse_h) * a.L_max + min(t * QT + lse_q, len - 1);
        st_lse = lse_u[at];
#pragma unroll
        for (int k = 1; k < kMaxKeyShares; ++k)
          if (k < a.lse_shares) st_more[k - 1] = (a.lse_of_share(k) + ubase * G)[at];
      }
    };
    if (t_first <= t_last) fetch(t_last, 0);
    __syncthreads();  // the previous block has finished with the tiles and what goes with them; odd_s is cleared
    Owned<DT, D> own;
    const bool odd_own = __builtin_amdgcn_ballot_w64(own.load(Kb, kj, len - 1)) != 0;
    float s1 = 0.0f, s2 = 0.0f;
    f32x16 pb[HEADS == 0 ? NSUB : 1];  // sums over the heads of a tile's probabilities

    int b = 0;
    for (int t = t_last; t >= t_first; --t) {
      for (int h = 0; h < (HEADS == 0 ? G : 1); ++h) {
        char* const tile = tiles[b];
        ++seq;
        if (st.store(tile) && DT == kF32) odd_s[b] = seq;
        if (threadIdx.x < P::TR) {
          if (a.lse_shares > 1) st_lse = merged_normaliser(st_lse, st_more, a.lse_shares);
          lse_s[b][threadIdx.x] = st_lse * a.lse_scale;
          if (count && HEADS == 1) rinv_s[b][threadIdx.x] = 1.0f / static_cast<float>(t * P::TR + static_cast<int>(threadIdx.x) + 1);
        }
        __syncthreads();
        if (HEADS == 0 && h + 1 < G) fetch(t, h + 1);
        else if (t > t_first) fetch(t - 1, 0);
        const bool odd = DT == kF32 && (odd_own || __builtin_amdgcn_readfirstlane(odd_s[b]) == seq);
#pragma unroll
        for (int i = 0; i < NSUB; ++i) {
          const int sub = part + PARTS * i;
          const int ib = t * QT + sub * QS;  // first query position of the sub-tile; its last one is ib + QS - 1
          if (ib + QS - 1 < kg || ib >= len) continue;  // no query of the sub-tile reaches the wave's keys
          f32x16 c;
          if (odd) {
            c = score_tile_plain<D>(
                [&](int i) {
                  int pos = ib + i, head = h;
                  if constexpr (HEADS > 1) {
                    GroupedRows<PER>::locate(i, pos, head);
                    pos += ib;
                  }
                  return Qu + (static_cast<size_t>(head) * a.L_max + min(pos, len - 1)) * P::IN_ROW;
                },
                Kb + static_cast<size_t>(min(kj, len - 1)) * P::IN_ROW);
          } else {
            c = score_tile<P::TR>(tile, sub, own);
          }
          const bool interior = ib + QS - 1 < len && ib >= kg + 31 + w;
          const float* lt = &lse_s[b][sub * 32];
          if constexpr (HEADS > 1) {
            if (interior) column_update_grouped<true, PER>(c, lt, sc, ib, half, kj, len, w, rb, a.pol, s1, s2);
            else column_update_grouped<false, PER>(c, lt, sc, ib, half, kj, len, w, rb, a.pol, s1, s2);
          } else if constexpr (HEADS == 0) {
            if (h == 0) pb[i] = f32x16{0};
            if (interior) column_probs<true>(c, lt, sc, ib, half, kj, len, w, rb, pb[i]);
            else column_probs<false>(c, lt, sc, ib, half, kj, len, w, rb, pb[i]);
            if (h == G - 1) {  // every head has been added
              float e1 = 0.0f, e2 = 0.0f;
              if (count) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                  const float p = pb[i][e] * inv_heads;
                  e1 += p;
                  e2 += p * static_cast<float>(ib + 8 * (e >> 2) + 4 * half + (e & 3) + 1) > 1.0f ? 1.0f : 0.0f;
                }
              } else {  // (the last-query score of kImpLast is written over the squares later: prefill_last_row)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                  const float p = pb[i][e] * inv_heads;
                  e1 += p;
                  e2 = fmaf(p, p, e2);
                }
              }
              s1 += e1;
              s2 += e2;
            }
          } else {
            const float* rt = &rinv_s[b][sub * 32];
            if (count) column_update<false, true>(c, lt, rt, sc, ib, half, kj, len, w, rb, s1, s2);
            else if (interior) column_update<true, false>(c, lt, rt, sc, ib, half, kj, len, w, rb, s1, s2);
            else column_update<false, false>(c, lt, rt, sc, ib, half, kj, len, w, rb, s1, s2);
          }
        }
        b ^= 1;
      }
    }
    s1 += __shfl_xor(s1, 32, kWave);
    s2 += __shfl_xor(s2, 32, kWave);
    if constexpr (PARTS > 1) {
      if (part > 0 && half == 0) { other[0][part - 1][32 * grp + lane] = s1; other[1][part - 1][32 * grp + lane] = s2; }
      __syncthreads();
      if (part == 0 && half == 0) {
#pragma unroll
        for (int o = 0; o < PARTS - 1; ++o) { s1 += other[0][o][32 * grp + lane]; s2 += other[1][o][32 * grp + lane]; }
      }
    }
    if (part == 0 && half == 0 && kj < len) { out1[ubase + kj] = s1; out2[ubase + kj] = s2; }
  }
}

// Four consecutive elements of a row of V.
template <int DT> __device__ __forceinline__ void load_values(const char* row, int at, float* v) {
  if constexpr (DT == kF32) {
    unpack16<kF32>(load16(row + at * 4), v);
  } else {
    const uint2 w = *reinterpret_cast<const uint2*>(row + at * 2);
    v[0] = __uint_as_float(w.x << 16); v[1] = __uint_as_float(w.x & 0xffff0000u);
    v[2] = __uint_as_float(w.y << 16); v[3] = __uint_as_float(w.y & 0xffff0000u);
  }
}

// ------------------------------------------------------------------------------------------------
// pass 1 with the attention output O_i = sum_j P[i,j] v_j (see prefill_rows_out_mfma for the operand layouts).  The
// probabilities are fp32 numbers and are taken apart into three planes: a bf16 V, which is one plane, takes three products
// of 32 keys (one, of bf16 probabilities, misrounds 40 % of the outputs where three misround 0.03 %; 32 units x 2048 tokens:
// whole call 106 us with one, 126 with three), an fp32 V, taken apart likewise, takes six.  Those six run on a chain of their
// own and are added to the output once, so an output component sees one rounding per 32 keys.
template <int DT, int D, int PARTS>
__global__ __launch_bounds__(kThreads, DT == kF32 && D == 128 ? 1 : 2) void prefill_rows_out_planes(PrefillArgs a) {
  using P = Planes<DT, D, kTileRowsSmall<DT, D, PARTS>>;
  constexpr int kOwn = Shares<PARTS>::kOwn, GROUPS = Shares<PARTS>::GROUPS;
  constexpr int NBUF = DT == kBF16 && PARTS < 4 ? 2 : 1;  // else one tile of K and V planes fills what two workgroups leave each other
  constexpr int DB = D / 32;
  __shared__ __attribute__((aligned(16))) char tilesK[NBUF][P::TILE];
  __shared__ __attribute__((aligned(16))) char tilesV[NBUF][P::TILEV];
  __shared__ float other[2][PARTS > 1 ? 2 * kWave : 1];
  __shared__ int odd_s[NBUF], odd_v[NBUF];  // see prefill_rows_planes
  int u, blk_id;
  if (!locate_heads(a.units, a.whole, a.group, a.pairs, u, blk_id)) return;
  const int uk = u / a.group;
  const int len = a.len[uk];
  const int n_blocks = (len + kOwn - 1) / kOwn;
  if (blk_id >= n_blocks) return;
  const int blk = n_blocks - 1 - blk_id;  // long rows first
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int half = lane >> 5, grp = wave % GROUPS, part = wave / GROUPS;
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  const size_t kbase = static_cast<size_t>(uk) * a.L_max;
  const char* Qb = static_cast<const char*>(a.Q) + ubase * P::IN_ROW;
  const char* Kb = static_cast<const char*>(a.K) + kbase * P::IN_ROW;
  const char* Vb = static_cast<const char*>(a.V) + kbase * P::IN_ROW;
  const float sc = a.scale_log2;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const int q0 = blk * kOwn;
  const int qw0 = q0 + 32 * grp;
  const int qi = qw0 + (lane & 31);
  if (threadIdx.x < NBUF) odd_s[threadIdx.x] = odd_v[threadIdx.x] = -1;
  Pieces<DT, D, P::TR> stK, stV;
  stK.load(Kb, 0, len - 1);
  stV.load(Vb, 0, len - 1);
  __syncthreads();
  Owned<DT, D> own;
  const bool odd_own = __builtin_amdgcn_ballot_w64(own.load(Qb, qi, len - 1)) != 0;
  float m = -INFINITY, l = 0.0f;
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = f32x16{0};
  // transpose reads of a V^T fragment: 16-lane group g reads columns 16 (g % 2) .. +15, key rows 4 (g / 2) .. +3
  const int i16 = lane & 15, g16 = lane >> 4;
  const int tr_off = ((g16 >> 1) * 4 + (i16 >> 2)) * P::ROWV + ((g16 & 1) * 16 + (i16 & 3) * 4) * 2;

  const int n_tiles = (min(len, q0 + kOwn) - 1) / P::TR + 1;
  for (int t = 0; t < n_tiles; ++t) {
    const int buf = NBUF == 2 ? t & 1 : 0;
    char* const tileK = tilesK[buf];
    char* const tileV = tilesV[buf];
    if (NBUF == 1 && t > 0) __syncthreads();  // everybody is done with the previous tile
    if (stK.store(tileK) && DT == kF32) odd_s[buf] = t;
    if (stV.store_values(tileV)) odd_v[buf] = t;
    __syncthreads();
    if (t + 1 < n_tiles) {
      stK.load(Kb, (t + 1) * P::TR, len - 1);
      stV.load(Vb, (t + 1) * P::TR, len - 1);
    }
    const bool odd = DT == kF32 && (odd_own || __builtin_amdgcn_readfirstlane(odd_s[buf]) == t);
    const bool odd_values = __builtin_amdgcn_readfirstlane(odd_v[buf]) == t;
#pragma unroll
    for (int i = 0; i < P::SUBS / PARTS; ++i) {
      const int sub = part + PARTS * i;
      const int kb = t * P::TR + sub * 32;
      if (kb > qw0 + 31) continue;  // wholly above the diagonal for every query of this wave
      f32x16 s;
      if (odd) s = score_tile_plain<D>([&](int i) { return Kb + static_cast<size_t>(min(kb + i, len - 1)) * P::IN_ROW; },
                                       Qb + static_cast<size_t>(min(qi, len - 1)) * P::IN_ROW);
      else s = score_tile<P::TR>(tileK, sub, own);
      // ---- probabilities against the reference m (lazily raised: see prefill_rows_out_mfma) and their sum
      const bool interior = kb + 31 + w <= qw0;
      float pv[16];
      float sum = 0.0f;
      bool done = false;
      if (interior && !odd_values) {
        const float neg = -m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          pv[r] = fast_exp2(fmaf(s[r], sc, neg));
          sum += pv[r];
        }
        done = __builtin_amdgcn_ballot_w64(!(sum <= 0x1p16f)) == 0;
      }
      if (!done) {
        float mb = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float x = s[r] * sc;
          if (!interior) {
            const int key = kb + 8 * (r >> 2) + 4 * half + (r & 3);
            if (w > 0 && qi - key < w) x += rb;
            if (key > qi) x = -INFINITY;
          }
          pv[r] = x;
          mb = fmaxf(mb, x);
        }
        mb = fmaxf(mb, __shfl_xor(mb, 32, kWave));  // both lane halves feed one matrix product: one reference
        const float m_new = fmaxf(m, mb);
        const float ref = m_new > -INFINITY ? m_new : 0.0f;  // no finite logit yet: every term is 2^-inf = 0
        if (__any(m_new > m)) {
          const float alpha = m_new > -INFINITY ? fast_exp2(m - m_new) : 1.0f;
          l *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        }
        m = m_new;
        sum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          pv[r] = fast_exp2(pv[r] - ref);
          sum += pv[r];
        }
      }
      l += sum;
      // ---- O^T += V^T . P^T
      if (odd_values) {  // V as it is, one key at a time, for the queries that see the key
#pragma unroll 1
        for (int key = 0; key < 32; ++key) {
          float mine = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; ++r) mine = (8 * (r >> 2) + (r & 3)) == (key & ~4) ? pv[r] : mine;
          const float pk = __shfl(mine, (lane & 31) + 32 * ((key >> 2) & 1), kWave);
          if (kb + key > qi || kb + key >= len) continue;
          const char* vr = Vb + static_cast<size_t>(kb + key) * P::IN_ROW;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
              float v[4];
              load_values<DT>(vr, db * 32 + 8 * g4 + 4 * half, v);
#pragma unroll
              for (int e = 0; e < 4; ++e) o[db][4 * g4 + e] = fmaf(pk, v[e], o[db][4 * g4 + e]);
            }
        }
        continue;
      }
      bf16x8 pf[3][2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        pf[0][r >> 3][r & 7] = static_cast<__bf16>(pv[r]);
        const float r1 = pv[r] - static_cast<float>(pf[0][r >> 3][r & 7]);
        pf[1][r >> 3][r & 7] = static_cast<__bf16>(r1);
        pf[2][r >> 3][r & 7] = static_cast<__bf16>(r1 - static_cast<float>(pf[1][r >> 3][r & 7]));
      }
      // two 16-key steps x DB blocks of 32 head dimensions
      auto values = [&](int plane, int ks, int db) {
        const char* vt = tileV + plane * P::PLANEV + (sub * 32 + ks * 16) * P::ROWV + tr_off + db * 64;
        const uint2 lo = lds_read_transposed(vt), hi = lds_read_transposed(vt + 8 * P::ROWV);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
      };
      auto p = [&](int plane, int ks) { return __builtin_bit_cast(uint4, pf[plane][ks]); };
      if constexpr (DT == kBF16) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          uint4 v[DB];
#pragma unroll
          for (int db = 0; db < DB; ++db) v[db] = values(0, ks, db);
#pragma unroll
          for (int plane = 2; plane >= 0; --plane)  // the small terms first
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] = mm(v[db], p(plane, ks), o[db]);
        }
      } else {
#pragma unroll
        for (int d2 = 0; d2 < DB; d2 += 2) {  // two chains at a time
          f32x16 c[2];
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {  // the small terms first, the hi x hi products last
            uint4 h[2], mid[2], lo[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              h[e] = values(0, ks, d2 + e);
              mid[e] = values(1, ks, d2 + e);
              lo[e] = values(2, ks, d2 + e);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(lo[e], p(0, ks), ks == 0 ? f32x16{0} : c[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(h[e], p(2, ks), c[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(mid[e], p(1, ks), c[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(mid[e], p(0, ks), c[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(h[e], p(1, ks), c[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) c[e] = mm(h[e], p(0, ks), c[e]);
          }
          o[d2] += c[0];
          o[d2 + 1] += c[1];
        }
      }
    }
  }
  l += __shfl_xor(l, 32, kWave);  // each lane half summed different keys of the same query
  // The parts hold sums over different keys of the same queries: the upper half of the waves hands its own to the lower half,
  // until one wave per group is left.
#pragma unroll
  for (int left = PARTS / 2; left > 0; left /= 2) {
    static_assert(PARTS == 1 || NBUF * P::TILE >= 2 * DB * 16 * kWave * 4, "the partners' outputs fit the K tiles");
    const int to = wave % (GROUPS * left);  // the wave that takes the sums of wave to + GROUPS * left
    float* const mo = reinterpret_cast<float*>(&tilesK[0][0]) + to * (DB * 16 * kWave) + lane;
    __syncthreads();  // everybody is done with the tiles, or with the sums handed over before
    if (part >= left && part < 2 * left) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) mo[(db * 16 + r) * kWave] = o[db][r];
      other[0][to * kWave + lane] = m;
      other[1][to * kWave + lane] = l;
    }
    __syncthreads();
    if (part >= left) continue;
    const float m1 = other[0][to * kWave + lane], l1 = other[1][to * kWave + lane];
    const float M = fmaxf(m, m1);
    // (a part that attended nothing has no sums; a weight that underflows still meets an infinite sum)
    const bool some0 = m > -INFINITY, some1 = m1 > -INFINITY;
    const float w0 = some0 ? fast_exp2(m - M) : 0.0f, w1 = some1 ? fast_exp2(m1 - M) : 0.0f;
    l = l * w0 + l1 * w1;
    m = M;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        o[db][r] = (some0 ? o[db][r] * w0 : 0.0f) + (some1 ? mo[(db * 16 + r) * kWave] * w1 : 0.0f);
  }
  if (part == 0 && qi < len) {
    if (half == 0) a.lse[ubase + qi] = m + log2f(l);
    const float inv = 1.0f / l;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const size_t at = (ubase + qi) * D + db * 32 + 8 * g4 + 4 * half;
        const float v0 = o[db][4 * g4] * inv, v1 = o[db][4 * g4 + 1] * inv, v2 = o[db][4 * g4 + 2] * inv, v3 = o[db][4 * g4 + 3] * inv;
        if constexpr (DT == kBF16) {
          *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.O) + at) =
              make_uint2(f32_to_bf16(v0) | (static_cast<uint32_t>(f32_to_bf16(v1)) << 16),
                         f32_to_bf16(v2) | (static_cast<uint32_t>(f32_to_bf16(v3)) << 16));
        } else {
          *reinterpret_cast<float4*>(static_cast<float*>(a.O) + at) = make_float4(v0, v1, v2, v3);
        }
      }
  }
}

// ------------------------------------------------------------------------------------------------
template <int DT, int D, int PARTS>
void launch_columns_of_group(const PrefillArgs& b, unsigned n, hipStream_t s) {
  switch (b.group) {
    case 1: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 1>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 2: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 2>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 3: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 3>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 4: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 4>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 5: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 5>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 6: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 6>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 7: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 7>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 8: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 8>), dim3(n), dim3(kThreads), 0, s, b); break;
    case 16: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 16>), dim3(n), dim3(kThreads), 0, s, b); break;
    default: hipLaunchKernelGGL((prefill_columns_planes<DT, D, PARTS, 0>), dim3(n), dim3(kThreads), 0, s, b); break;
  }
}

// Workgroups of the passes that a compute unit holds (fp32 / 128 with two parts: one).
template <int DT, int D> constexpr int kResident = D == 128 ? 2 : DT == kBF16 ? 4 : 3;

template <int DT, int D>
void launch_rows(const PrefillArgs& a, const PassPlan& plan, hipStream_t s) {
  ProfScope ps(kProfPrefillRows, s);
  PrefillArgs b = a;
  b.pairs = plan.ids; b.paired = plan.paired; b.ksplit = plan.split;
  const int ids = a.group * plan.ids * plan.split;
  b.whole = mfma::units_on_whole_dies(a.units, ids, kResident<DT, D>);
  const dim3 grid(mfma::workgroup_ids(a.units, b.whole, ids));
  switch (plan.parts) {
    case 1: hipLaunchKernelGGL((prefill_rows_planes<DT, D, 1>), grid, dim3(kThreads), 0, s, b); break;
    case 2: if constexpr (D == 64 || DT == kBF16) hipLaunchKernelGGL((prefill_rows_planes<DT, D, 2>), grid, dim3(kThreads), 0, s, b); break;
    default: if constexpr (DT == kBF16) hipLaunchKernelGGL((prefill_rows_planes<DT, D, 4>), grid, dim3(kThreads), 0, s, b); break;
  }
  if (plan.split > a.lse_shares) launch_merge_key_shares(b, s);
}

// The row pass with output takes single blocks.  Whole call, us, 64 owned rows (two waves share 32) against 128: bf16 / 64
// 4 x 1024 tokens 44 / 54, 32 x 2048 117 / 134, 256 x 2048 589 / 619, but 1024 x 256 126 / 116; fp32 / 64 4 x 1024 78 / 97,
// 128 x 1024 253 / 255, but 256 x 1024 478 / 455, 256 x 2048 1588 / 1433 and 1024 x 256 246 / 206.  Row pass, us: 32 owned rows
// against 64 for bf16 / 64 1 x 4575 60 / 86, but 16 streams x 4396 194 / 163; 64 against 128 for fp32 / 128 7 x 2578 172 / 247,
// but with more than one of its workgroups, which do not share a compute unit, 108 x 129 42 / 27.
// Left-over units that share dies are streamed through one die's L2 together.  The fp32 output pass, one or two workgroups per
// compute unit, does not hide what then misses it: with long prompts five or more left over are worth the idle dies (5 units x 2
// heads x 4000 tokens of fp32 / 128 1018 us shared, 690 whole; 43 prompts of 5, 13, 21 and 29 units: geometric mean 1.04, between
// 0.98 and 1.48).  Three behind others are not: 11 x 2 x 2000 0.89, 19 x 2 x 2000 0.92.
inline bool shared_units_miss_the_l2(int units, long long unit_bytes) { return unit_bytes >= (3 << 19) && (units & 7) >= 5; }

template <int DT, int D>
void launch_rows_out(const PrefillArgs& a, hipStream_t s) {
  ProfScope ps(kProfPrefillRows, s);
  PrefillArgs b = a;
  b.paired = 0; b.ksplit = 1;
  const long long streams = static_cast<long long>(a.units) * a.group;
  int parts = D == 64 ? 2 : streams * ceil_div(a.L_max, 64) <= 300 ? 2 : 1;
  if (DT == kBF16 && streams * ceil_div(a.L_max, 64) < 512 && a.L_max > 384) parts = 4;
  b.pairs = ceil_div(a.L_max, 128 / parts);
  b.whole = mfma::units_on_whole_dies(a.units, a.group * b.pairs, D == 128 ? 1 : DT == kBF16 && parts == 2 ? 3 : 2);
  if (DT == kF32 && shared_units_miss_the_l2(a.units, 2ll * a.L_max * D * 4)) b.whole = (a.units + 7) & ~7;
  const dim3 grid(mfma::workgroup_ids(a.units, b.whole, a.group * b.pairs));
  switch (parts) {
    case 1: if constexpr (D == 128) hipLaunchKernelGGL((prefill_rows_out_planes<DT, D, 1>), grid, dim3(kThreads), 0, s, b); break;
    case 2: hipLaunchKernelGGL((prefill_rows_out_planes<DT, D, 2>), grid, dim3(kThreads), 0, s, b); break;
    default: if constexpr (DT == kBF16) hipLaunchKernelGGL((prefill_rows_out_planes<DT, D, 4>), grid, dim3(kThreads), 0, s, b); break;
  }
}

template <int DT, int D>
void launch_columns(PrefillArgs& a, const PassPlan& plan, hipStream_t s) {
  ProfScope ps(kProfPrefillColumns, s);
  PrefillArgs b = a;
  b.pairs = plan.ids; b.paired = plan.paired; b.qsplit = plan.split;
  if (a.lse_given != nullptr) { b.lse = const_cast<float*>(a.lse_given); b.lse_scale = kLog2e; }  // read, never written here
  const int ids = plan.ids * plan.split;
  b.whole = mfma::units_on_whole_dies(a.units, ids, DT == kF32 && D == 128 && plan.parts == 2 ? 1 : kResident<DT, D>);
  const unsigned n = mfma::workgroup_ids(a.units, b.whole, ids);
  switch (plan.parts) {
    case 1: launch_columns_of_group<DT, D, 1>(b, n, s); break;
    case 2: launch_columns_of_group<DT, D, 2>(b, n, s); break;
    default: if constexpr (DT == kBF16) launch_columns_of_group<DT, D, 4>(b, n, s); break;
  }
  join_query_shares(a, b, s);
}

template <int DT, int D>
hipError_t launch_t(PrefillArgs& a, hipStream_t s) {
  const PassPlan columns = plan_columns(DT, D, a.units, a.group, a.L_max, a.shares);
  if (!a.skip_rows) {
    if (prefill_rows_are_tiny(a, DT == kF32, D)) launch_prefill_rows_simple(DT, D, a, s);
    else if (a.O != nullptr) launch_rows_out<DT, D>(a, s);
    else {
      const PassPlan rows = plan_rows(DT, D, a.units, a.group, a.L_max, a.row_shares());
      columns_merge_normalisers(a, rows, columns);
      launch_rows<DT, D>(a, rows, s);
    }
  }
  launch_columns<DT, D>(a, columns, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_attention_planes(int dtype, int head_dim, PrefillArgs& a, hipStream_t s) {
  if (dtype == kF32 && head_dim == 64) return launch_t<kF32, 64>(a, s);
  if (dtype == kF32 && head_dim == 128) return launch_t<kF32, 128>(a, s);
  if (dtype == kBF16 && head_dim == 64) return launch_t<kBF16, 64>(a, s);
  return hipErrorInvalidValue;
}
// bf16 / 128: the passes for which their plan does not ask for the kernels of prefill_mfma.hip
void launch_prefill_rows_planes_wide(const PrefillArgs& a, const PassPlan& plan, hipStream_t s) { launch_rows<kBF16, 128>(a, plan, s); }
void launch_prefill_columns_planes_wide(PrefillArgs& a, const PassPlan& plan, hipStream_t s) { launch_columns<kBF16, 128>(a, plan, s); }

}  // namespace roco
