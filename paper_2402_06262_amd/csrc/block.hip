// Block-wise evict-and-encode on gfx950 (section 5.3 "Overhead" and appendix B of the paper: the number of
// tokens freed and encoded within one eviction step is a block size b; b = 1 is the token-wise scheme).
//
// With n tokens cached, E = max(0, n + b - B) tokens are evicted in one step (E single evictions by the rule of
// section 4.3 with frozen statistics = the E lowest mean attention scores among the s + E - 1 lowest variances),
// the block's tokens go in order to the ascending list of freed and still-empty slots, query i of the block
// attends every retained token and the block's tokens 0..i, and every attended token gets p, p^2 and 1 added to
// its statistics.  The point of the scheme is that K and V are streamed once per block instead of once per token:
// the step stays HBM-bound, so encoding b tokens costs about what encoding one does.
//
//   block_prepare : one workgroup per unit.  Victims (two exact radix selects), ordered slot assignment,
//                   K / V rows of the block written into their slots, pos / statistics of those slots reset.
//   block_attend  : grid (splits, units), two waves.  Each wave streams 32-slot tiles of K and V through LDS of its
//                   own and scores them against the block's queries on the matrix cores (score tile = K . Q^T, the
//                   query in the lane; one or two tiles of 32 query rows, every K and V^T fragment read from LDS
//                   feeding both), stores the base-2 logits, keeps an online softmax per query and accumulates
//                   O^T = V^T . P^T with V^T fragments from the LDS transpose read.
//   block_attend_shared : the same for fp32 and head_dim 64, on the vector ALUs (see there).
//   block_finish  : one workgroup per unit.  Merges the partials per query, writes the outputs, adds the
//                   statistics of all rows to every slot and chooses the victim a following single-token step
//                   would take.
//
// Steps of bf16 mostly take one or two kernels that keep the logits on the compute unit instead (block_fused.hpp).
//
// The same three kernels serve grouped-query attention (section 5.3, "Extension to Grouped-Query Attention"):
// g query heads share the unit's keys and values, the query rows are (token, head) pairs, and the statistics
// receive, once per token, the mean of its g heads' probabilities (BlockArgs::heads).
#include <cstdlib>

#include "block_steps.hpp"
#include "profile.hpp"

namespace roco {
namespace {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"

using namespace mfma;

constexpr int kPrepThreads = 1024;  // 512 when the units outnumber the compute units (see launch_block)
constexpr int kAttThreads = 128;  // two waves: every other 32-slot tile each
constexpr int kFinThreads = 1024;
constexpr int kQ = 32;            // query rows per matrix tile
static_assert(kMaxBlock == 2 * kQ, "a step holds at most two tiles of query rows");

// ------------------------------------------------------------------------------------------------
// LDS: the ranking keys are in LDS (B <= kMaxDecodeBudgetLds), here and in block_finish.
template <int NT, bool LDS>
__global__ __launch_bounds__(NT, 8) void block_prepare(BlockArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds_keys[];  // [2][B] when B <= kMaxDecodeBudgetLds
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<1>::kWords];
  __shared__ uint32_t scan_sh[NT / kWave + 1];
  __shared__ int slot_of[kMaxBlock];
  const int u = blockIdx.x, tid = threadIdx.x;
  const int B = a.B, b = a.block;
  const int n = a.n_used[u];
  float* acc = a.stats + static_cast<size_t>(u) * 3 * B;
  float* acc2 = acc + B;
  float* cnt = acc2 + B;
  int32_t* bidx = a.blk_idx + static_cast<size_t>(u) * B;
  uint32_t* const var_key = LDS ? lds_keys : a.keys + static_cast<size_t>(u) * 2 * B;
  uint32_t* const mas_key = var_key + B;

  take_slots<NT, 1, true>(a, u, n, var_key, mas_key, sel_sh, scan_sh, slot_of, [&](int j, int bi) {
    if (bi >= 0) {
      acc[j] = 0.0f;
      acc2[j] = 0.0f;
      cnt[j] = 0.0f;
    }
    bidx[j] = bi;
  });
  if (tid == 0) a.n_used[u] = min(B, n + b);
}

// ------------------------------------------------------------------------------------------------
// K and V of a wave: 32 slots a tile, two tiles of each in LDS, private to the wave and filled by loads that go straight there
// (tile_ring.hpp), so that nothing but the wave's own load counter orders the stream: no barrier, no staging registers, and the
// buffer of an operand is requested again as soon as its tile has been used.  At least three operand tiles of a wave are on
// their way at any time, 96 KiB per compute unit.  64-slot tiles staged through registers, with a barrier per tile and nothing in
// flight between the arrival of a tile and the requests after the barrier, took 55.9 us where this takes 51.1 (233 units x 3
// heads x 1644 slots), 54.5 / 49.1 (136 x 4 heads x 14 tokens x 1096), 183.9 / 174.4 (415 x 35 tokens x 2640), 125.2 / 123.8 at
// 512 x 16 tokens x 2048, whose 64 MiB of logits cost 30 us between the reads.
// K chunk c of row r lies in slot c ^ (r & 15), V chunk c in slot c ^ 4 (r & 3): see TileRing and OutRing.
struct WaveTiles {
  static constexpr int kSlots = 32;
  static constexpr int kOperand = kSlots * kRowBytes;  // 8 KiB
  static constexpr int kBytes = 4 * kOperand;          // K, K, V, V of one wave
  static constexpr int kLoads = kOperand / 1024;       // wave-wide loads per operand tile
};
// NQT: tiles of 32 query rows (1 or 2).  The workspace planes are addressed with a.qrows = 32 NQT rows per unit.
// WINDOW: a recency bias is in force (the slots' positions come along with the K tiles).
template <int NQT, bool STREAMING, bool WINDOW>
__global__ __launch_bounds__(kAttThreads) void block_attend(BlockArgs a) {
  using T = WaveTiles;
  constexpr int QR = NQT * kQ;
  constexpr int kSideLoads = WINDOW ? 2 : 1;  // block indices of a K tile's slots, and their positions
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];  // the two waves' tiles; reused for the merge
  __shared__ __attribute__((aligned(256))) int32_t bidx_s[2][2][kWave], pos_s[WINDOW ? 2 : 1][2][kWave];  // [wave][buffer]
  __shared__ float merge_m[QR], merge_l[QR];
  const int u = blockIdx.y, split = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int half = lane >> 5, qi = lane & 31;  // this lane's query row inside a tile
  const int B = a.B, b = a.queries;
  // Usually block_prepare has run: n_used counts the block's tokens and their rows are in the cache.  A single-token
  // step skips it (BlockArgs::single): the token's slot is known from the state, its row is read from k_new / v_new
  // and written into the cache by the wave that streams that slot, as in the token-wise decode kernels.
  int n = a.n_used[u];
  int fresh = -1;
  if (a.single) {
    const bool was_full = n >= B;
    fresh = was_full ? min(max(a.next_slot[u], 0), B - 1) : n;
    n = was_full ? B : n + 1;
  }
  const int row0 = split * a.rows_per_split;
  const int row1 = min(n, row0 + a.rows_per_split);
  const size_t pidx = static_cast<size_t>(u) * a.splits + split;
  char* Kb = static_cast<char*>(a.K) + static_cast<size_t>(u) * B * kRowBytes;
  char* Vb = static_cast<char*>(a.V) + static_cast<size_t>(u) * B * kRowBytes;
  float* z = a.z + static_cast<size_t>(u) * QR * B;
  const float sc = a.scale_log2;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const int qp0 = a.qpos0[u];
  int ti[NQT], qp[NQT];  // this lane's block token per tile; the heads of a group share its position
#pragma unroll
  for (int t2 = 0; t2 < NQT; ++t2) {
    ti[t2] = (kQ * t2 + qi) / a.heads;
    qp[t2] = qp0 + ti[t2];
  }

  // The split's rows: slots past the unit's last one come back as zeros (and are masked below).  A descriptor's size and offsets
  // have 32 bits, which the rows of a split fit (kMaxSplitRows), not those of a unit.
  const uint32_t split_bytes = static_cast<uint32_t>(max(row1 - row0, 0)) * kRowBytes;
  const v4i32 kbuf = make_buffer(Kb + static_cast<size_t>(row0) * kRowBytes, split_bytes);
  const v4i32 vbuf = make_buffer(Vb + static_cast<size_t>(row0) * kRowBytes, split_bytes);
  const v4i32 bbuf = make_buffer(a.blk_idx + static_cast<size_t>(u) * B, static_cast<uint32_t>(B) * 4u);
  const v4i32 pbuf = make_buffer(a.pos + static_cast<size_t>(u) * B, static_cast<uint32_t>(B) * 4u);
  char* const my_tiles = lds_dyn + wave * T::kBytes;
  const uint32_t tiles_addr = lds_address(my_tiles);
  const uint32_t bidx_addr = lds_address(&bidx_s[wave][0][0]), pos_addr = lds_address(&pos_s[WINDOW ? wave : 0][0][0]);
  // This lane's chunks of a tile, rows 4 i + lane / 16.  All of a row's offset inside the tile is the lane's: the scalar offset is the
  // tile's first row, which exists, so that rows behind the last one are out of range by the lane's offset alone (see load16_to_lds).
  int koff[T::kLoads], voff[T::kLoads];
#pragma unroll
  for (int i = 0; i < T::kLoads; ++i) {
    const int r = 4 * i + (lane >> 4);
    koff[i] = r * kRowBytes + (((lane & 15) ^ (r & 15)) << 4);
    voff[i] = r * kRowBytes + (((lane & 15) ^ ((r & 3) << 2)) << 4);
  }
  // The wave's tiles: every other one of the split, from a start that differs between workgroups, so that workgroups running
  // side by side do not walk the memory channels in lock step (the online softmax does not care about the order).
  const int n_tiles = row1 > row0 ? (row1 - row0 + T::kSlots - 1) / T::kSlots : 0;
  const int mine = (n_tiles - wave + 1) / 2;
  const int rot = mine > 0 ? static_cast<int>((static_cast<unsigned>(u) * 5u + static_cast<unsigned>(split) * 3u) %
                                              static_cast<unsigned>(mine))
                           : 0;
  auto tile_row = [&](int t) { return row0 + (2 * (t + rot < mine ? t + rot : t + rot - mine) + wave) * T::kSlots; };
  auto request_k = [&](int t) {
    const int row = tile_row(t);
    const uint32_t dst = tiles_addr + (t & 1) * T::kOperand;
    const int soff = __builtin_amdgcn_readfirstlane((row - row0) * kRowBytes);
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) load16_to_lds_hint<STREAMING>(kbuf, dst + i * 1024, koff[i], soff);
    const int side = __builtin_amdgcn_readfirstlane(row * 4);
    load4_to_lds(bbuf, bidx_addr + (t & 1) * (kWave * 4), lane * 4, side);
    if (WINDOW) load4_to_lds(pbuf, pos_addr + (t & 1) * (kWave * 4), lane * 4, side);
  };
  auto request_v = [&](int t) {
    const uint32_t dst = tiles_addr + (2 + (t & 1)) * T::kOperand;
    const int soff = __builtin_amdgcn_readfirstlane((tile_row(t) - row0) * kRowBytes);
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) load16_to_lds_hint<STREAMING>(vbuf, dst + i * 1024, voff[i], soff);
  };

  // B operand: the block's queries (lanes beyond the block reuse its last query; their results are dropped)
  uint4 own[NQT][kKSteps];
#pragma unroll
  for (int t2 = 0; t2 < NQT; ++t2) {
    const char* qrow = static_cast<const char*>(a.q) + (static_cast<size_t>(u) * b + min(kQ * t2 + qi, b - 1)) * kRowBytes;
#pragma unroll
    for (int kk = 0; kk < kKSteps; ++kk) own[t2][kk] = load16(qrow + kk * 32 + half * 16);
  }
  if (mine > 0) { request_k(0); request_v(0); }
  if (mine > 1) { request_k(1); request_v(1); }
  float m[NQT], l[NQT];
  f32x16 o[NQT][4];
#pragma unroll
  for (int t2 = 0; t2 < NQT; ++t2) {
    m[t2] = -INFINITY;
    l[t2] = 0.0f;
#pragma unroll
    for (int db = 0; db < 4; ++db) o[t2][db] = f32x16{0};
  }
  // fragment reads: K row lane % 32, chunk 2 kk + half; V transposed, rows 4 half + (lane % 16) / 4 (+ 8), the lane's 8 bytes of
  // columns 32 db + 16 (lane / 16 % 2) + 4 (lane % 4)
  const int kfrag = (lane & 31) * kRowBytes + ((half ^ (lane & 15)) << 4);
  int vfrag[4];
  {
    const int rr = (lane & 15) >> 2;
#pragma unroll
    for (int db = 0; db < 4; ++db)
      vfrag[db] = (4 * half + rr) * kRowBytes + ((db ^ rr) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  }
  // The new token's row of a single-token step, put over the old one in the tile and in the cache: 16 lanes.
  auto put_row = [&](const void* rows, char* cache, char* tile, int slot_in_tile, int swizzle) {
    if (lane < 16) {
      const uint4 row = load16(static_cast<const char*>(rows) + static_cast<size_t>(u) * kRowBytes + lane * 16);
      *reinterpret_cast<uint4*>(tile + slot_in_tile * kRowBytes + ((lane ^ swizzle) << 4)) = row;
      *reinterpret_cast<uint4*>(cache + static_cast<size_t>(fresh) * kRowBytes + lane * 16) = row;
    }
  };

  for (int t = 0; t < mine; ++t) {
    char* const tileK = my_tiles + (t & 1) * T::kOperand;
    char* const tileV = my_tiles + (2 + (t & 1)) * T::kOperand;
    const int sb = tile_row(t);  // first slot of the tile
    const bool holds_fresh = fresh >= sb && fresh < sb + T::kSlots;
    // K(t) has landed; V(t), and K and V of the next tile, may still be on their way (and logits stored since, which the
    // counter holds too: then a little more than K(t) has landed)
    if (t + 1 < mine) wait_loads<3 * T::kLoads + kSideLoads>();
    else wait_loads<T::kLoads>();
    if (holds_fresh) {
      put_row(a.k_new, Kb, tileK, fresh - sb, (fresh - sb) & 15);
      if (WINDOW && lane == 0) pos_s[WINDOW ? wave : 0][t & 1][fresh - sb] = qp0;
    }
    // ---- scores of 32 slots x 32 NQT queries: every K fragment feeds one accumulator chain per query tile
    f32x16 sacc[NQT];
    {
      const f32x16 zero = {0};
#pragma unroll
      for (int kk = 0; kk < kKSteps; ++kk) {
        const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tileK + (kfrag ^ (kk << 5))));
#pragma unroll
        for (int t2 = 0; t2 < NQT; ++t2)
          sacc[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, __builtin_bit_cast(bf16x8, own[t2][kk]),
                                                             kk == 0 ? zero : sacc[t2], 0, 0, 0);
      }
    }
    // index and position of the lane's 16 slots
    int biv[16], psv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int base = 8 * g4 + 4 * half;  // index inside the tile of 4 consecutive slots
      const int4 bi = *reinterpret_cast<const int4*>(&bidx_s[wave][t & 1][base]);
      biv[4 * g4] = bi.x; biv[4 * g4 + 1] = bi.y; biv[4 * g4 + 2] = bi.z; biv[4 * g4 + 3] = bi.w;
      if (WINDOW) {
        const int4 ps = *reinterpret_cast<const int4*>(&pos_s[WINDOW ? wave : 0][t & 1][base]);
        psv[4 * g4] = ps.x; psv[4 * g4 + 1] = ps.y; psv[4 * g4 + 2] = ps.z; psv[4 * g4 + 3] = ps.w;
      }
    }
    reads_done();
    if (t + 2 < mine) request_k(t + 2);
    bf16x8 pfrag[NQT][2];
#pragma unroll
    for (int t2 = 0; t2 < NQT; ++t2) {
    // ---- base-2 logits: a slot is visible if it exists and does not hold a later token of the block
    const int q = kQ * t2 + qi;
    float tv[16];
    float mb = -INFINITY;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int slot0 = sb + 8 * g4 + 4 * half;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x = sacc[t2][4 * g4 + e] * sc;
        if (WINDOW) {
          const int dlt = qp[t2] - psv[4 * g4 + e];
          if (dlt >= 0 && dlt < w) x += rb;
        }
        if (slot0 + e >= row1 || (!a.single && biv[4 * g4 + e] > ti[t2])) x = -INFINITY;
        tv[4 * g4 + e] = x;
        mb = fmaxf(mb, x);
      }
      if (q < b && slot0 < row1) {  // logits of real queries and real slots are kept for the statistics
        *reinterpret_cast<float4*>(z + static_cast<size_t>(q) * B + slot0) =
            make_float4(tv[4 * g4], tv[4 * g4 + 1], tv[4 * g4 + 2], tv[4 * g4 + 3]);
      }
    }
    mb = fmaxf(mb, __shfl_xor(mb, 32, kWave));  // both lane halves feed one matrix product
    const float m_new = fmaxf(m[t2], mb);
    if (__any(m_new > m[t2])) {
      const float alpha = (m_new > -INFINITY) ? fast_exp2(m[t2] - m_new) : 1.0f;
      l[t2] *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t2][db][r] *= alpha;
    }
    m[t2] = m_new;
    float sum = 0.0f;
    const float ref = (m_new > -INFINITY) ? m_new : 0.0f;  // nothing visible yet: every term is 2^-inf = 0
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float pv = fast_exp2(tv[r] - ref);
      sum += pv;
      pfrag[t2][r >> 3][r & 7] = static_cast<__bf16>(pv);
    }
    l[t2] += sum;
    }
    // ---- O^T += V^T . P^T: V(t) has landed; K and V of the next tile, and K of the one after, may be on their way
    if (t + 2 < mine) wait_loads<3 * T::kLoads + 2 * kSideLoads>();
    else if (t + 1 < mine) wait_loads<2 * T::kLoads + kSideLoads>();
    else wait_loads<0>();
    if (holds_fresh) put_row(a.v_new, Vb, tileV, fresh - sb, ((fresh - sb) & 3) << 2);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const char* vt = tileV + ks * (16 * kRowBytes);
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const uint2 lo = lds_read_transposed(vt + vfrag[db]);
        const uint2 hi = lds_read_transposed(vt + 8 * kRowBytes + vfrag[db]);
        const bf16x8 afrag = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
        for (int t2 = 0; t2 < NQT; ++t2)
          o[t2][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, pfrag[t2][ks], o[t2][db], 0, 0, 0);
      }
    }
    reads_done();
    if (t + 2 < mine) request_v(t + 2);
  }
#pragma unroll
  for (int t2 = 0; t2 < NQT; ++t2) l[t2] += __shfl_xor(l[t2], 32, kWave);  // the lane halves summed different slots

  // ---- merge the two waves (wave 1 hands its state to wave 0 through LDS), then write the split's partial
  __syncthreads();  // everybody is done with the tiles
  float* mo = reinterpret_cast<float*>(lds_dyn);  // [QR query rows][128 dims]
  if (wave == 1) {
#pragma unroll
    for (int t2 = 0; t2 < NQT; ++t2) {
      const int q = kQ * t2 + qi;
      if (half == 0) { merge_m[q] = m[t2]; merge_l[q] = l[t2]; }
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) mo[q * D + db * 32 + 8 * (r >> 2) + 4 * half + (r & 3)] = o[t2][db][r];
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int t2 = 0; t2 < NQT; ++t2) {
      const int q = kQ * t2 + qi;
      if (q >= b) continue;  // lanes beyond the step's query rows repeated its last query: nothing of theirs is kept
      const float m1 = merge_m[q], l1 = merge_l[q];
      const float M = fmaxf(m[t2], m1);
      const float w0 = (m[t2] > -INFINITY) ? fast_exp2(m[t2] - M) : 0.0f;
      const float w1 = (m1 > -INFINITY) ? fast_exp2(m1 - M) : 0.0f;
      if (half == 0) {
        a.part_m[pidx * QR + q] = M;
        a.part_l[pidx * QR + q] = l[t2] * w0 + l1 * w1;
      }
      float* po = a.part_o + (pidx * QR + q) * D;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int d0 = db * 32 + 8 * g4 + 4 * half;
          float4 r4;
          const float4 other = (w1 > 0.0f) ? *reinterpret_cast<const float4*>(mo + q * D + d0)
                                           : make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // wave 1 saw nothing: ignore LDS
          r4.x = o[t2][db][4 * g4 + 0] * w0 + other.x * w1;
          r4.y = o[t2][db][4 * g4 + 1] * w0 + other.y * w1;
          r4.z = o[t2][db][4 * g4 + 2] * w0 + other.z * w1;
          r4.w = o[t2][db][4 * g4 + 3] * w0 + other.w * w1;
          *reinterpret_cast<float4*>(po + d0) = r4;
        }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// The attention of the block-wise / grouped-query step for the shapes the matrix-core kernel is not built for
// (fp32, head_dim 64), on the vector ALUs: grid (splits, units), four waves.  K and V are streamed once for all
// query rows of the step, as on the matrix-core path: a tile of 64 slots goes through LDS (as fp32), then
//   scores : a wave takes every fourth query row.  Its lanes form QS groups; a lane owns QS slots of the tile (one
//            lane of every group per slot) and the queries of its group, so that every K or Q value read from LDS
//            feeds several multiply-adds (a register block of QS slots x QL queries per lane: with one slot per
//            lane the broadcast reads of Q, not the arithmetic, set the pace).  The group keeps an online softmax
//            per query row (maximum and sum over the tile by lane reductions inside the group), stores the base-2
//            logits and leaves the tile's probabilities and the factor that rescales the running output in LDS.
//   output : a thread owns four output dimensions of every NG-th query row: O[q][d] = O[q][d] alpha[q] +
//            sum_r P[q][r] V[r][d], four slots at a time (one 16-byte read of P per row, of V per slot).
// The vector work grows with the number of query rows while the bytes do not: a step of many rows is bound by the
// ALUs, and still reads the cache once instead of once per row.  Produces what block_attend produces.
template <int D> struct SharedTile {
  static constexpr int kRows = 64;        // slots per tile
  static constexpr int kStride = D + 4;   // floats per K row in LDS: lanes that read consecutive rows hit different banks
  static size_t lds_bytes(int qmax) {     // K tile, V tile, probabilities, queries, rescale factors
    return (static_cast<size_t>(kRows) * kStride + static_cast<size_t>(kRows) * D + static_cast<size_t>(qmax) * kRows +
            static_cast<size_t>(qmax) * D + qmax) * sizeof(float);
  }
};

// QMAX: most query rows the instantiation takes (8, 16, 32 or 64).  The smaller ones need fewer registers and less LDS,
// so more workgroups fit a compute unit, and they keep two tiles in flight per workgroup instead of one.
// SINGLE: a single-token step without block_prepare (BlockArgs::single).  What it needs besides is kept out of the other steps'
// kernels, whose registers decide how many workgroups a compute unit holds: in one kernel for both, bf16 / 64 with 32 rows took
// 207 instead of 166, two workgroups instead of three (551 units x 1488 slots x 17 tokens 350 us against 252).  The single-token
// kernels of bf16 / 64 for 16 and 32 rows are held to three workgroups too (300 units x 744 slots x 16 heads 56.2 us, 66.5 with
// two; x 24 heads 73.7, 99.0 with two).
template <int DT, int D, int QMAX, bool SINGLE>
__global__ __launch_bounds__(256, (D != 64 ? 1 : DT == kBF16 && (QMAX == 16 || QMAX == 32) ? 3 : 2)) void block_attend_shared(BlockArgs a) {
  using G = RowGeom<DT, D>;
  using T = SharedTile<D>;
  constexpr int TR = T::kRows, KS = T::kStride, WAVES = 4;
  constexpr int KQ = QMAX / WAVES;       // query rows per wave: wave + 4 k
  constexpr int QS = KQ >= 4 ? 4 : KQ;   // lane groups of a wave = slots per lane
  constexpr int RG = kWave / QS;         // lanes per group; lane rg owns slots rg + RG i, i < QS
  constexpr int QL = KQ / QS;            // query rows per lane: k = qs + QS jq
  constexpr int DQ = D / 4;              // output phase: threads per query row, four dimensions each
  constexpr int NG = 256 / DQ;           // ... and groups of threads: group og takes rows og + NG k
  constexpr int OQ = QMAX >= NG ? QMAX / NG : 1;
  constexpr int CH = TR * G::LPR / 256;  // 16-byte pieces of a tile per thread and operand
  constexpr int PF = (QMAX <= 8 || (QMAX <= 32 && D == 64)) ? 2 : 1;  // tiles in flight
  static_assert(CH >= 1 && TR * G::LPR % 256 == 0, "a tile is dealt evenly to the threads");
  static_assert(QMAX % WAVES == 0 && KQ % QS == 0 && QS * RG == kWave && RG * QS == TR && QMAX <= kMaxBlock, "query rows and slots are dealt evenly");
  extern __shared__ __attribute__((aligned(16))) float lds_f[];
  __shared__ int32_t bidx_s[TR], pos_s[TR];
  float* const Kt = lds_f;                 // [TR][KS]
  float* const Vt = Kt + TR * KS;          // [TR][D]
  float* const Pt = Vt + TR * D;           // [QMAX][TR] probabilities of the tile against the running reference
  float* const Qs = Pt + QMAX * TR;        // [QMAX][D]  queries times scale * log2(e)
  float* const al = Qs + QMAX * D;         // [QMAX]     factor for the running output of a query row
  const int u = blockIdx.y, split = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int B = a.B, nq = a.queries, QR = a.qrows;  // QR: rows per unit of the workspace planes
  // block_prepare has run: the block's rows are in the cache and counted -- or it is a single-token step without it, as in block_attend
  int n = a.n_used[u];
  int fresh = -1;
  if constexpr (SINGLE) {
    const bool was_full = n >= B;
    fresh = was_full ? min(a.next_slot[u], B - 1) : n;
    if (fresh < 0) {  // (the tiles are not in use yet)
      uint32_t* const sel_sh = reinterpret_cast<uint32_t*>(lds_f);
      fresh = victim_by_statistics<256, 1>(a.stats + static_cast<size_t>(u) * 3 * B, a.pos + static_cast<size_t>(u) * B, B, a.pol, a.scope,
                                        sel_sh, reinterpret_cast<uint2*>(sel_sh + SelectLds<1>::kWords));
      __syncthreads();
    }
    if (split == 0 && tid == 0) a.blk_idx[static_cast<size_t>(u) * B] = fresh;  // for block_finish
    n = was_full ? B : n + 1;
  }
  const int row0 = split * a.rows_per_split;
  const int row1 = min(n, row0 + a.rows_per_split);
  const size_t pidx = static_cast<size_t>(u) * a.splits + split;
  char* const Kb = static_cast<char*>(a.K) + static_cast<size_t>(u) * B * G::ROW_BYTES;
  char* const Vb = static_cast<char*>(a.V) + static_cast<size_t>(u) * B * G::ROW_BYTES;
  const int32_t* bidx = a.blk_idx + static_cast<size_t>(u) * B;
  const int32_t* pos = a.pos + static_cast<size_t>(u) * B;
  float* z = a.z + static_cast<size_t>(u) * QR * B;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const int qp0 = a.qpos0[u];

  for (int idx = tid; idx < QMAX * G::LPR; idx += 256) {  // the step's queries, scaled, as fp32; zeros beyond them
    const int q = idx / G::LPR, c = idx % G::LPR;
    float f[G::EPL];
    unpack16<DT>(load16(static_cast<const char*>(a.q) + (static_cast<size_t>(u) * nq + min(q, nq - 1)) * G::ROW_BYTES + c * 16), f);
#pragma unroll
    for (int e = 0; e < G::EPL; ++e) Qs[q * D + c * G::EPL + e] = q < nq ? f[e] * a.scale_log2 : 0.0f;
  }

  const int rg = lane % RG, qs = lane / RG;
  int qrow[QL];        // this lane's query rows (may lie beyond the step's: those compute on zeros and store nothing)
  float m[QL], l[QL];  // their online softmax (the same in every lane of the group)
#pragma unroll
  for (int jq = 0; jq < QL; ++jq) {
    qrow[jq] = wave + WAVES * (qs + QS * jq);
    m[jq] = -INFINITY;
    l[jq] = 0.0f;
  }
  const int dq = tid % DQ, og = tid / DQ;
  float4 o[OQ];
#pragma unroll
  for (int k = 0; k < OQ; ++k) o[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

  const int n_tiles = row1 > row0 ? (row1 - row0 + TR - 1) / TR : 0;
  uint4 pk[PF][CH], pv[PF][CH];
  int32_t st_bidx[PF], st_pos[PF];  // first wave: of slot `lane` of the tiles on their way
  auto fetch = [&](int t, uint4* fk, uint4* fv, int32_t& fb, int32_t& fp) {
    const int tr0 = row0 + t * TR;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int idx = tid + 256 * i;
      const int row = min(tr0 + idx / G::LPR, n - 1);  // rows past the end are dealt with below
      const size_t off = static_cast<size_t>(row) * G::ROW_BYTES + (idx % G::LPR) * 16;
      fk[i] = a.streaming ? load16_streaming(Kb + off) : load16(Kb + off);
      fv[i] = a.streaming ? load16_streaming(Vb + off) : load16(Vb + off);
    }
    if (tid < TR) {
      const int slot = min(tr0 + tid, n - 1);
      fb = SINGLE ? -1 : bidx[slot];
      fp = SINGLE && slot == fresh ? qp0 : pos[slot];
    }
  };
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    st_bidx[j] = -1;
    st_pos[j] = 0;
    if (j < n_tiles) fetch(j, pk[j], pv[j], st_bidx[j], st_pos[j]);
  }
  for (int t0 = 0; t0 < n_tiles; t0 += PF) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int t = t0 + j;
      if (t >= n_tiles) break;
      const int tr0 = row0 + t * TR;
      if (SINGLE && fresh >= tr0 && fresh < min(tr0 + TR, row1)) {  // a single token's row takes its slot, here and in the cache
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int idx = tid + 256 * i, col = (idx % G::LPR) * 16;
          if (tr0 + idx / G::LPR == fresh) {
            pk[j][i] = load16(static_cast<const char*>(a.k_new) + static_cast<size_t>(u) * G::ROW_BYTES + col);
            pv[j][i] = load16(static_cast<const char*>(a.v_new) + static_cast<size_t>(u) * G::ROW_BYTES + col);
            *reinterpret_cast<uint4*>(Kb + static_cast<size_t>(fresh) * G::ROW_BYTES + col) = pk[j][i];
            *reinterpret_cast<uint4*>(Vb + static_cast<size_t>(fresh) * G::ROW_BYTES + col) = pv[j][i];
          }
        }
      }
      // Rows behind the last slot are copies of one (their loads only had to stay in range), and that one may be the slot which a
      // single token fills for the first time, whose bytes are arbitrary, or whose infinite value it overwrites: as V they are
      // zeros, since a weight of 0 does not silence NaN or infinity.  (Scores of such rows are replaced, whatever they are.  In the
      // other steps block_prepare has written that slot.)
      if (SINGLE && tr0 + TR > row1) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
          if (tr0 + (tid + 256 * i) / G::LPR >= row1) pv[j][i] = make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int idx = tid + 256 * i;
        const int r = idx / G::LPR, c = idx % G::LPR;
        float fk[G::EPL], fv[G::EPL];
        unpack16<DT>(pk[j][i], fk);
        unpack16<DT>(pv[j][i], fv);
#pragma unroll
        for (int e = 0; e < G::EPL; e += 4) {
          *reinterpret_cast<float4*>(Kt + r * KS + c * G::EPL + e) = make_float4(fk[e], fk[e + 1], fk[e + 2], fk[e + 3]);
          *reinterpret_cast<float4*>(Vt + r * D + c * G::EPL + e) = make_float4(fv[e], fv[e + 1], fv[e + 2], fv[e + 3]);
        }
      }
      if (tid < TR) { bidx_s[tid] = st_bidx[j]; pos_s[tid] = st_pos[j]; }
      __syncthreads();  // the tile (and, the first time, the queries) are in LDS
      if (t + PF < n_tiles) fetch(t + PF, pk[j], pv[j], st_bidx[j], st_pos[j]);

      // ---- scores: QS slots x QL query rows per lane (a wave whose first query row lies beyond the step's has none)
      if (wave < nq) {
      float part[QS][QL];
#pragma unroll
      for (int i = 0; i < QS; ++i)
#pragma unroll
        for (int jq = 0; jq < QL; ++jq) part[i][jq] = 0.0f;
#pragma unroll 2  // (fully unrolled, the compiler hoists every LDS read of the tile and runs out of registers)
      for (int c0 = 0; c0 < D; c0 += 8) {
        float4 kc[QS][2];
#pragma unroll
        for (int i = 0; i < QS; ++i) {
          kc[i][0] = *reinterpret_cast<const float4*>(Kt + (rg + RG * i) * KS + c0);
          kc[i][1] = *reinterpret_cast<const float4*>(Kt + (rg + RG * i) * KS + c0 + 4);
        }
#pragma unroll
        for (int jq = 0; jq < QL; ++jq) {
          const int q = min(qrow[jq], QMAX - 1);
          const float4 qa = *reinterpret_cast<const float4*>(Qs + q * D + c0);
          const float4 qb = *reinterpret_cast<const float4*>(Qs + q * D + c0 + 4);
#pragma unroll
          for (int i = 0; i < QS; ++i) {
            float s = part[i][jq];
            s = fmaf(kc[i][0].x, qa.x, s); s = fmaf(kc[i][0].y, qa.y, s);
            s = fmaf(kc[i][0].z, qa.z, s); s = fmaf(kc[i][0].w, qa.w, s);
            s = fmaf(kc[i][1].x, qb.x, s); s = fmaf(kc[i][1].y, qb.y, s);
            s = fmaf(kc[i][1].z, qb.z, s); s = fmaf(kc[i][1].w, qb.w, s);
            part[i][jq] = s;
          }
        }
      }
#pragma unroll
      for (int jq = 0; jq < QL; ++jq) {
        const int q = qrow[jq];
        const bool live = q < nq;   // uniform inside a group of lanes, not inside the wave
        const int ti = q / a.heads;  // the heads of a group share the token's position
        float x[QS];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < QS; ++i) {
          const int r = rg + RG * i, slot = tr0 + r;
          float v = part[i][jq];
          const int dlt = qp0 + ti - pos_s[r];
          if (w > 0 && dlt >= 0 && dlt < w) v += rb;
          if (slot >= row1 || bidx_s[r] > ti) v = -INFINITY;  // no such slot, or a later token of the block
          if (live && slot < row1) z[static_cast<size_t>(q) * B + slot] = v;  // kept for the statistics
          x[i] = v;
          mx = fmaxf(mx, v);
        }
        const float m_new = fmaxf(m[jq], group_max<RG>(mx));
        const float ref = (m_new > -INFINITY) ? m_new : 0.0f;  // nothing visible yet: every term is 2^-inf = 0
        const float alpha = (m_new > -INFINITY) ? fast_exp2(m[jq] - m_new) : 1.0f;
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < QS; ++i) {
          const float pr = fast_exp2(x[i] - ref);
          sum += pr;
          if (live) Pt[q * TR + rg + RG * i] = pr;
        }
        l[jq] = fmaf(l[jq], alpha, group_sum<RG>(sum));
        m[jq] = m_new;
        if (live && rg == 0) al[q] = alpha;
      }
      }
      __syncthreads();  // the tile's probabilities are in LDS

      // ---- O[q][d] = O[q][d] alpha[q] + sum_r P[q][r] V[r][d] (a wave whose first query row is beyond the step's: idle)
      if ((wave * kWave) / DQ < nq) {
#pragma unroll
      for (int k = 0; k < OQ; ++k) {
        const int q = og + NG * k;
        if (q < nq) {
          const float f = al[q];
          o[k].x *= f; o[k].y *= f; o[k].z *= f; o[k].w *= f;
        }
      }
      for (int r = 0; r < TR; r += 4) {
        const float4 v0 = *reinterpret_cast<const float4*>(Vt + r * D + 4 * dq);
        const float4 v1 = *reinterpret_cast<const float4*>(Vt + (r + 1) * D + 4 * dq);
        const float4 v2 = *reinterpret_cast<const float4*>(Vt + (r + 2) * D + 4 * dq);
        const float4 v3 = *reinterpret_cast<const float4*>(Vt + (r + 3) * D + 4 * dq);
#pragma unroll
        for (int k = 0; k < OQ; ++k) {
          const int q = og + NG * k;
          if (q < nq) {
            const float4 p4 = *reinterpret_cast<const float4*>(Pt + q * TR + r);
            o[k].x = fmaf(p4.x, v0.x, o[k].x); o[k].y = fmaf(p4.x, v0.y, o[k].y);
            o[k].z = fmaf(p4.x, v0.z, o[k].z); o[k].w = fmaf(p4.x, v0.w, o[k].w);
            o[k].x = fmaf(p4.y, v1.x, o[k].x); o[k].y = fmaf(p4.y, v1.y, o[k].y);
            o[k].z = fmaf(p4.y, v1.z, o[k].z); o[k].w = fmaf(p4.y, v1.w, o[k].w);
            o[k].x = fmaf(p4.z, v2.x, o[k].x); o[k].y = fmaf(p4.z, v2.y, o[k].y);
            o[k].z = fmaf(p4.z, v2.z, o[k].z); o[k].w = fmaf(p4.z, v2.w, o[k].w);
            o[k].x = fmaf(p4.w, v3.x, o[k].x); o[k].y = fmaf(p4.w, v3.y, o[k].y);
            o[k].z = fmaf(p4.w, v3.z, o[k].z); o[k].w = fmaf(p4.w, v3.w, o[k].w);
          }
        }
      }
      }
      __syncthreads();  // everybody is done with the tile before the next one overwrites it
    }
  }

  // ---- this split's partial: reference, sum and unnormalised output per query row
#pragma unroll
  for (int jq = 0; jq < QL; ++jq) {
    const int q = qrow[jq];
    if (q < nq && rg == 0) {
      a.part_m[pidx * QR + q] = m[jq];
      a.part_l[pidx * QR + q] = l[jq];
    }
  }
#pragma unroll
  for (int k = 0; k < OQ; ++k) {
    const int q = og + NG * k;
    if (q < nq) *reinterpret_cast<float4*>(a.part_o + (pidx * QR + q) * D + 4 * dq) = o[k];
  }
}

// ------------------------------------------------------------------------------------------------
// One workgroup per unit: it walks all slots of the unit two per thread and sweep, keeps the ranking keys in LDS and
// chooses the next victim itself.  (Spreading the update over slot chunks and selecting in a launch of its own
// measured slower for every number of query rows: the extra launch costs more than the longer sweep.)
// R: logits of this many query rows are loaded at a time.  A larger R hides more of their latency in a longer loop body,
// which has to be fetched first (a launch starts with a cold instruction cache): of 2 / 4 / 8, 64 rows of 4 heads on 128 units
// took 51 / 46 / 44 us, 16 rows of one head on 512 units 28.7 / 29.7 / 30.5.
template <int DT, int D, int R, bool LDS>
__global__ __launch_bounds__(kFinThreads, 8) void block_finish(BlockArgs a) {
  constexpr int NT = kFinThreads;
  constexpr int kSlots = 2 * NT;  // slots per sweep
  constexpr bool kMatrix = DT == kBF16 && D == 128;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds_keys[];  // [2][B] ranking keys when B <= kMaxDecodeBudgetLds
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<1>::kWords];
  __shared__ uint2 best_sh[NT / kWave];
  __shared__ float2 norm[kMaxBlock];  // reference and 1 / sum of every query row
  // the merge of the splits is done before the search begins
  float2* const part_ml = reinterpret_cast<float2*>(sel_sh);                        // [kBlockPartials]
  float* const weight = reinterpret_cast<float*>(part_ml + kBlockPartials);  // ditto
  static_assert(3 * kBlockPartials <= SelectLds<1>::kWords, "the merge fits the search's words");
  const int u = blockIdx.x, tid = threadIdx.x;
  const int B = a.B, nq = a.queries, S = a.splits, QR = a.qrows;
  int n = a.n_used[u];
  int fresh = -1;  // single-token step without block_prepare: the slot the token took, which this kernel books
  bool evicted = false;
  if (a.single) {
    evicted = n >= B;
    // (behind block_attend_shared: the slot it has chosen)
    fresh = !kMatrix ? a.blk_idx[static_cast<size_t>(u) * B] : evicted ? min(max(a.next_slot[u], 0), B - 1) : n;
    n = evicted ? B : n + 1;
  }
  const int heads = a.heads;
  const float inv_heads = 1.0f / static_cast<float>(heads);
  const float* pm = a.part_m + static_cast<size_t>(u) * S * QR;
  const float* pl = a.part_l + static_cast<size_t>(u) * S * QR;
  const float* po = a.part_o + static_cast<size_t>(u) * S * QR * D;

  // The splits' normalisers of a query row come in with one load per (split, row) and are merged from LDS in split order;
  // a loop of dependent trips to memory per row would cost more than the rest of the merge.
  static_assert(kBlockPartials <= NT, "one thread per (split, row)");
  const int my_row = tid & (QR - 1);  // (split, row) in the order of the planes
  const bool merges = tid < S * QR && my_row < nq;
  float2 mine = make_float2(-INFINITY, 0.0f);
  if (merges) {
    mine = make_float2(pm[tid], pl[tid]);
    part_ml[tid] = mine;
  }
  __syncthreads();
  if (merges) {
    float M = -INFINITY, L = 0.0f;
#pragma unroll 1
    for (int i = my_row; i < S * QR; i += QR) M = fmaxf(M, part_ml[i].x);
#pragma unroll 1
    for (int i = my_row; i < S * QR; i += QR) {
      const float2 ml = part_ml[i];
      L += (ml.x > -INFINITY) ? ml.y * fast_exp2(ml.x - M) : 0.0f;
    }
    // (a split that attended nothing has no partials; a weight that underflows still meets an infinite partial)
    weight[tid] = (mine.x > -INFINITY) ? fast_exp2(mine.x - M) : -1.0f;
    if (tid < nq) norm[tid] = make_float2(M, 1.0f / L);
  }
  __syncthreads();  // every thread has read n_used and next_slot
  if (a.single && tid == 0) {
    int32_t* pos = a.pos + static_cast<size_t>(u) * B;
    const int old_pos = pos[fresh];
    pos[fresh] = a.qpos0[u];
    a.n_used[u] = n;
    if (a.evicted_slot) a.evicted_slot[u] = evicted ? fresh : -1;
    if (a.evicted_pos) a.evicted_pos[u] = evicted ? old_pos : -1;
  }
  // outputs: the partials of eight splits of an element are requested together
#pragma unroll 1
  for (int idx = tid; idx < nq * D; idx += NT) {
    const int q = idx / D, dd = idx % D;
    float o = 0.0f;
#pragma unroll 1
    for (int s0 = 0; s0 < S; s0 += 8) {
      float part[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (s0 + i < S) part[i] = po[(static_cast<size_t>(s0 + i) * QR + q) * D + dd];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (s0 + i < S) {
          const float wgt = weight[(s0 + i) * QR + q];
          o += wgt < 0.0f ? 0.0f : part[i] * wgt;
        }
      }
    }
    store_elem<DT>(a.out, (static_cast<size_t>(u) * nq + q) * D + dd, o * norm[q].y);
  }
  // statistics: every slot receives, per block token that attended it, the head-mean of the probabilities
  float* acc = a.stats + static_cast<size_t>(u) * 3 * B;
  float* acc2 = acc + B;
  float* cnt = acc2 + B;
  const float* z = a.z + static_cast<size_t>(u) * QR * B;
  const bool full = n >= B;
  uint32_t* const var_key = LDS ? lds_keys : a.keys + static_cast<size_t>(u) * 2 * B;
  uint32_t* const mas_key = var_key + B;
  const bool by_pos = a.pol.needs_pos();
  const bool squares = !a.pol.keeps_last_score() && !a.pol.counts_above_average();
  // B is a multiple of 4 on this path, so a pair of slots is inside [0, B).
#pragma unroll 1
  for (int j = tid * 2; j < n; j += kSlots) {
  const int2 bi = a.single ? make_int2(-1, -1)
                                       : *reinterpret_cast<const int2*>(a.blk_idx + static_cast<size_t>(u) * B + j);
  const float2 a1 = *reinterpret_cast<const float2*>(acc + j);
  const float2 a2 = *reinterpret_cast<const float2*>(acc2 + j);
  const float2 cc = *reinterpret_cast<const float2*>(cnt + j);
  float s1[2] = {a1.x, a1.y}, s2[2] = {a2.x, a2.y}, sc[2] = {cc.x, cc.y};
  const int biv[2] = {bi.x, bi.y};
#pragma unroll
  for (int e = 0; e < 2; ++e)
    if (j + e == fresh) { s1[e] = 0.0f; s2[e] = 0.0f; sc[e] = 0.0f; }  // the new token starts from zero
  // The query rows (token-major, a token's heads side by side) are taken R at a time.
  float mean[2] = {0.0f, 0.0f};  // sum over the query heads of the token under way of p
  int t = 0, h = 0;
#pragma unroll 1
  for (int q0 = 0; q0 < nq; q0 += R) {
    float2 zz[R];
#pragma unroll
    for (int i = 0; i < R; ++i)
      zz[i] = *reinterpret_cast<const float2*>(z + static_cast<size_t>(min(q0 + i, nq - 1)) * B + j);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (q0 + i < nq) {
        const float2 mi = norm[q0 + i];
        mean[0] += fast_exp2(zz[i].x - mi.x) * mi.y;
        mean[1] += fast_exp2(zz[i].y - mi.x) * mi.y;
        if (++h == heads) {  // the token's last head: its head-mean goes to the slots it attended
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            if (j + e < n && biv[e] <= t) {  // older tokens have index -1: attended by every row
              const float p = mean[e] * inv_heads;  // group-wise averaged probability (exact for one head)
              s1[e] += p;
              s2[e] = squares ? s2[e] + p * p : a.pol.second_statistic(s2[e], p, static_cast<float>(n - a.block + t + 1));
              sc[e] += 1.0f;
            }
            mean[e] = 0.0f;
          }
          h = 0;
          ++t;
        }
      }
    }
  }
  *reinterpret_cast<float2*>(acc + j) = make_float2(s1[0], s1[1]);
  *reinterpret_cast<float2*>(acc2 + j) = make_float2(s2[0], s2[1]);
  *reinterpret_cast<float2*>(cnt + j) = make_float2(sc[0], sc[1]);
  if (full) {  // then both are slots of the unit
    int pv[2] = {0, 0};
    if (by_pos) {
#pragma unroll
      for (int e = 0; e < 2; ++e) pv[e] = j + e == fresh ? a.qpos0[u] : a.pos[static_cast<size_t>(u) * B + j + e];
    }
    uint2 mk, vk;
    ranking_keys<2>(s1, s2, sc, pv, a.pol, &mk.x, &vk.x);
    *reinterpret_cast<uint2*>(mas_key + j) = mk;
    *reinterpret_cast<uint2*>(var_key + j) = vk;
  }
  }
  // the victim a following single-token step would take
  if (full) {
    __syncthreads();
    const int victim = select_victim_block<NT, 1>(var_key, mas_key, B, a.pol, a.scope, sel_sh, best_sh);
    if (tid == 0) a.next_slot[u] = victim;
  } else if (tid == 0) {
    a.next_slot[u] = -1;
  }
}

}  // namespace

// ROCO_BLOCK_SINGLE=0 keeps block_prepare in single-token steps (tests run both).
static bool single_step_off() {
  const char* e = getenv("ROCO_BLOCK_SINGLE");
  return e != nullptr && e[0] == '0';
}

template <int DT, int D, int R>
void launch_block_finish(const BlockArgs& a, hipStream_t s) {
  const size_t key_lds = key_lds_bytes(a.B);
  // (if the limit is refused, the launch fails and is reported)
  (void)allow_key_lds(reinterpret_cast<const void*>(block_finish<DT, D, R, true>), key_lds);
  if (key_lds != 0) hipLaunchKernelGGL((block_finish<DT, D, R, true>), dim3(a.units), dim3(kFinThreads), key_lds, s, a);
  else hipLaunchKernelGGL((block_finish<DT, D, R, false>), dim3(a.units), dim3(kFinThreads), 0, s, a);
}
template <int DT, int D>
void launch_block_tail(const BlockArgs& a, hipStream_t s) {
  ProfScope ps(kProfBlockFinish, s);
  if (a.queries > 32) launch_block_finish<DT, D, 8>(a, s);
  else if (a.heads > 1) launch_block_finish<DT, D, 4>(a, s);
  else launch_block_finish<DT, D, 2>(a, s);
}

template <int DT, int D, int QMAX, bool SINGLE>
hipError_t launch_block_shared_t(const BlockArgs& a, hipStream_t s) {
  const size_t lds = SharedTile<D>::lds_bytes(QMAX);  // 37 to 114 KiB: the limit is set on every call
  const void* fn = reinterpret_cast<const void*>(block_attend_shared<DT, D, QMAX, SINGLE>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((block_attend_shared<DT, D, QMAX, SINGLE>), dim3(a.splits, a.units), dim3(256), lds, s, a);
  return hipSuccess;
}
template <int DT, int D, int QMAX>
hipError_t launch_block_shared_q(const BlockArgs& a, hipStream_t s) {
  return a.single ? launch_block_shared_t<DT, D, QMAX, true>(a, s) : launch_block_shared_t<DT, D, QMAX, false>(a, s);
}

template <int DT, int D>
hipError_t launch_block_shared(const BlockArgs& a, hipStream_t s) {
  {
    ProfScope ps(kProfBlockAttend, s);
    const hipError_t e = a.queries <= 8    ? launch_block_shared_q<DT, D, 8>(a, s)
                         : a.queries <= 16 ? launch_block_shared_q<DT, D, 16>(a, s)
                         : a.queries <= 32 ? launch_block_shared_q<DT, D, 32>(a, s)
                                           : launch_block_shared_q<DT, D, kMaxBlock>(a, s);
    if (e != hipSuccess) return e;
  }
  launch_block_tail<DT, D>(a, s);
  return hipSuccess;
}

template <int NQT, bool STREAMING, bool WINDOW>
hipError_t launch_block_attend_t(const BlockArgs& a, hipStream_t s) {
  constexpr size_t kLds = 2 * WaveTiles::kBytes;  // 64 KiB, and what the kernel declares: above the default limit; set on every call
  const void* fn = reinterpret_cast<const void*>(block_attend<NQT, STREAMING, WINDOW>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kLds)) != hipSuccess)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((block_attend<NQT, STREAMING, WINDOW>), dim3(a.splits, a.units), dim3(kAttThreads), kLds, s, a);
  return hipSuccess;
}
hipError_t launch_block_attend(const BlockArgs& a, hipStream_t s) {
  ProfScope ps(kProfBlockAttend, s);
  const bool two = a.qrows > kQ, window = a.recency_window > 0;
  if (a.streaming) {
    if (window) return two ? launch_block_attend_t<2, true, true>(a, s) : launch_block_attend_t<1, true, true>(a, s);
    return two ? launch_block_attend_t<2, true, false>(a, s) : launch_block_attend_t<1, true, false>(a, s);
  }
  if (window) return two ? launch_block_attend_t<2, false, true>(a, s) : launch_block_attend_t<1, false, true>(a, s);
  return two ? launch_block_attend_t<2, false, false>(a, s) : launch_block_attend_t<1, false, false>(a, s);
}

// dtype / head_dim other than bf16 / 128 take the vector-ALU attention
hipError_t launch_block(int dtype, int head_dim, const BlockArgs& args, hipStream_t s) {
  BlockArgs a = args;
  // A single-token step needs no block_prepare (steps with / without it, us: 8 heads on 1 unit x 2340 slots of bf16 / 64 39.5 /
  // 27.8, 2 heads on 140 x 3252 of fp32 / 128 142 / 135).
  a.single = (a.block == 1 && !single_step_off()) ? 1 : 0;
  const size_t key_lds = key_lds_bytes(a.B);
  if (!allow_key_lds(reinterpret_cast<const void*>(block_prepare<512, true>), key_lds) ||
      !allow_key_lds(reinterpret_cast<const void*>(block_prepare<kPrepThreads, true>), key_lds))
    return hipErrorInvalidValue;
  const bool mfma_path = dtype == kBF16 && head_dim == 128;
  hipError_t fused;
  const bool prepared = a.block == 1 && !a.single;  // is asked for
  if (dtype == kBF16 && !prepared && launch_block_fused(head_dim, a, s, fused)) return fused != hipSuccess ? fused : hipGetLastError();
  if (!a.single) {
    ProfScope ps(kProfBlockPrepare, s);
    // Two 1024-thread workgroups do not run side by side on a compute unit here (measured: the second half of 512
    // units starts when the first has finished); with more units than compute units 512 threads are faster.
    const dim3 grid(a.units);
    if (key_lds == 0) hipLaunchKernelGGL((block_prepare<kPrepThreads, false>), grid, dim3(kPrepThreads), 0, s, a);
    else if (a.units > 256) hipLaunchKernelGGL((block_prepare<512, true>), grid, dim3(512), key_lds, s, a);
    else hipLaunchKernelGGL((block_prepare<kPrepThreads, true>), grid, dim3(kPrepThreads), key_lds, s, a);
  }
  if (mfma_path) {
    if (launch_block_attend(a, s) != hipSuccess) return hipErrorInvalidValue;
    launch_block_tail<kBF16, 128>(a, s);
  } else {
    hipError_t e = hipErrorInvalidValue;
    if (dtype == kBF16 && head_dim == 64) e = launch_block_shared<kBF16, 64>(a, s);
    else if (dtype == kF32 && head_dim == 64) e = launch_block_shared<kF32, 64>(a, s);
    else if (dtype == kF32 && head_dim == 128) e = launch_block_shared<kF32, 128>(a, s);
    if (e != hipSuccess) return e;
  }
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  return hipSuccess;
}

}  // namespace roco
