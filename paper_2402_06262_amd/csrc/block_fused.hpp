// The whole step of a unit in one workgroup, for bf16: block-wise evict-and-encode and grouped single tokens whose logits stay
// on the compute unit.
//
// The three kernels of block.hip pass the logits through memory, because the statistics need every row's normaliser, which is known
// when the last slot has been seen: 4 bytes per slot and row out and back in, beside the 512 bytes of the slot's key and value, and
// each launch begins when the last workgroup of the one before has ended.  Here one workgroup does a unit's whole step and keeps its
// logits in registers:
//   K           streamed once, the logits of a wave's tiles into its registers
//   eviction    of several tokens (take_slots); before K or after it
//   normalisers the waves' maxima, then sums, through LDS; the registers then hold probabilities
//   statistics  the probabilities go to LDS, where the tiles were; every thread adds the rows of its slots, and the next victim is chosen
//   outputs     V streamed once against the registers.  Probabilities are taken as sums of bf16 numbers (split_positive): the matrix
//               cores idle.  Two for head_dim 128, where rounded to one they made half of the output's error (2.1e-3 against 64 bits,
//               1.7e-3 so); three for head_dim 64, whose three kernels multiply all 24 bits on the vector ALUs
// 33 to 64 rows, and 25 to 32 over more than 1024 slots of head_dim 128: two workgroups per unit, each with half of the tokens (HALVES).  Both stream
// K and V, which one of them finds in their die's L2, and both evict, alike; they leave their sums of probabilities and squares to
// block_book, which adds them to the statistics and does what depends on or changes the state that both have read (128 units x 2048 x
// 16 tokens of 4 heads 95 -> 65 us).
//
// V is only waited for by the outputs, and nothing waits for them: every other group of eight units streams K before it evicts and V
// before its statistics, so that on the whole some workgroups use the memory while others rank (512 units x 2048 slots x 16 tokens:
// 125 us with one order for all, 118 with turns at the eviction, 111 with both).
//
// What bounds it: a compute unit takes 49 GB/s alone, 41 when half of the chip's units do (5.2 TB/s), 24 when all do (6.1 TB/s), so a
// workgroup per unit streams as fast as several once the units cover half of the chip: 128 x 4 heads x 2048 slots 45.9 -> 37.6 us (26
// of them the stream, 4 the search for the next victim), 512 x 16 tokens x 2048 163 -> 109 (88 the stream).
// A launch begins with a cold instruction cache, and what is fetched once costs a third of a microsecond per KiB: chains over all of a
// wave's tiles only move registers, everything else is done once, on the tile moved.
#pragma once
#include <algorithm>

#include "block_steps.hpp"
#include "profile.hpp"

namespace roco {
namespace fused {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"

using mfma::bf16x8;
using mfma::lds_address;
using mfma::lds_read_transposed;
using mfma::load16_to_lds_hint;
using mfma::load4_to_lds;
using mfma::make_buffer;
using mfma::reads_done;
using mfma::v4i32;
using mfma::wait_loads;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileSlots = 32;  // slots of a tile of K or V: one wave's
constexpr int kQ16 = 16;         // query rows per matrix tile

// Geometry of bf16 rows of HD elements.
template <int HD> struct Rows {
  static constexpr int kBytes = 2 * HD;
  static constexpr int kChunks = kBytes / 16;             // 16-byte chunks: lanes per row of a load
  static constexpr int kPerLoad = kWave / kChunks;        // rows of a wave-wide load
  static constexpr int kTile = kTileSlots * kBytes;       // bytes of a tile
  static constexpr int kLoads = kTile / 1024;             // wave-wide loads of a tile
  static constexpr int kSteps = HD / 32, kBlocks = HD / 16;  // of the matrix instruction: k-steps of a score, blocks of dimensions
  static constexpr int kOut = HD + 4;                     // floats per row of a wave's output in LDS
  static constexpr int kPlanes = HD == 128 ? 2 : 3;       // bf16 numbers of a probability
  // K chunk c of row r lies in slot c ^ swizzle_k(r), V chunk c in slot c ^ swizzle_v(r): 16 lanes that read a chunk of K of 16 rows,
  // and 32 that read 32 bytes of V of 8 rows, fall on distinct banks (256 bytes: two rows of 64 elements, one of 128).
  static __device__ __forceinline__ int swizzle_k(int r) { return HD == 128 ? r & 15 : (r >> 1) & 7; }
  static __device__ __forceinline__ int swizzle_v(int r) { return HD == 128 ? ((r & 3) << 2) ^ (((r >> 2) & 1) << 1) : ((r >> 1) & 3) << 1; }
};

// The 16x16x32 instruction as used here: lane l supplies row (l % 16) and the 8 consecutive k-elements from 8 (l / 16) on, for A and
// for B alike; register r of the result belongs to A-row 4 (l / 16) + r and B-row (l % 16).  Scores: A = 16 slots of K, B = the
// queries, so that a lane holds four consecutive slots of one query.  Output: A = V^T (16 dimensions), B = P^T; the eight slots
// that a lane supplies are the four it holds of either half of the tile, in both operands.
__device__ __forceinline__ f32x4 mfma16(const uint4& x, const uint4& y, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
}

// (fmaxf quiets its operands first: two instructions where this is half a one)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Eight probabilities as sums of N bf16 numbers: to within 2^-16 of each for two of them, exactly for three (but for bits below 2^-133).
// All of them are above zero where the probability is: each but the last is the largest bf16 number below what those before it leave
// over, the last at least the smallest of all.  So an infinite value keeps its sign in every product; rounded to the nearest, half of
// the remainders are zero or negative, and inf - inf or 0 inf is NaN.
template <int N>
__device__ __forceinline__ void split_positive(const f32x4 (&p)[2], uint4 (&planes)[N]) {
  uint32_t word[N][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float left = p[e >> 2][e & 3];
    const uint32_t least = min(__float_as_uint(left), 0x10000u);  // of a nonzero number; (fp32 has bf16's exponents)
#pragma unroll
    for (int i = 0; i < N - 1; ++i) {
      const uint32_t below = (max(__float_as_uint(left), 1u) - 1u) & 0xffff0000u;
      left -= __uint_as_float(below);
      word[i][e] = max(below, least);
    }
    word[N - 1][e] = max(__float_as_uint(left), least);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (N == 2 && i == 1) {
      bf16x8 r;
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = static_cast<__bf16>(__uint_as_float(word[i][e]));
      planes[i] = __builtin_bit_cast(uint4, r);
    } else {  // bf16 numbers already: the upper halves of the words
      const auto pair = [&](int e) { return __builtin_amdgcn_perm(word[i][e + 1], word[i][e], 0x07060302u); };
      planes[i] = make_uint4(pair(0), pair(2), pair(4), pair(6));
    }
  }
}

// Where half `h` of a unit's tokens leaves its sums of probabilities and, behind them, of their squares.
__device__ __forceinline__ float* part_sums(const BlockArgs& a, int u, int h) { return a.z + (static_cast<size_t>(u) * 2 + h) * 2 * a.B; }

// W waves.  NQ tiles of 16 query rows.  ZT: tiles of a wave whose logits its registers hold (32 W ZT slots in all).
// SINGLE: one token; its slot is known from the state.  lds_slots: slots whose probabilities the LDS takes at a time, a multiple of 32 W,
// four to a thread.  v_room: there is room for the first tiles of V beside them.
template <int HD, int W, int NQ, int ZT, bool SINGLE, bool STREAMING, bool WINDOW, bool HALVES = false>
__global__ __launch_bounds__(W * kWave, 2) void block_fused(BlockArgs a, int lds_slots, int v_room) {
  using R = Rows<HD>;
  constexpr int NT = W * kWave;
  constexpr int QR = NQ * kQ16;
  constexpr int kRowBytes = R::kBytes, kTileBytes = R::kTile, kTileLoads = R::kLoads;
  constexpr int kSide = WINDOW ? 1 : 0;  // the positions of a K tile's slots come along
  constexpr int PER_WORD = W == 4 ? 2 : 1;
  constexpr bool TURNS = ZT > 4 && NQ == 1;  // little to stream, or no registers to spare: the code for both orders costs more than they gain
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // two tiles of every wave; or ranking keys and probabilities; or the waves' outputs
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<PER_WORD>::kWords];
  __shared__ uint32_t scan_sh[W + 1];
  __shared__ uint2 best_sh[W];
  __shared__ int slot_of[kMaxBlock];
  __shared__ __attribute__((aligned(256))) int32_t pos_s[WINDOW ? W : 1][2][kWave];
  __shared__ float m_s[W][QR], l_s[W][QR];
  __shared__ float new_s[SINGLE ? 1 : QR][SINGLE ? 1 : HALVES ? kMaxBlock : QR];  // base-2 logits of the block's own tokens
  __shared__ __attribute__((aligned(16))) signed char bidx_s[SINGLE ? 16 : 32 * W * ZT];  // block token that a slot holds, or -1
  const int u = !HALVES ? blockIdx.x : (blockIdx.x >> 4 << 3) + (blockIdx.x & 7);  // a unit's halves share a die's L2
  if (HALVES && u >= a.units) return;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int qi = lane & 15, g = lane >> 4;
  const int B = a.B, heads = a.heads;
  const int tok0 = HALVES && (blockIdx.x & 8) != 0 ? (a.block + 1) / 2 : 0;  // this workgroup's tokens
  const int toks = !HALVES ? a.block : tok0 != 0 ? a.block - tok0 : (a.block + 1) / 2;
  const int nq = HALVES ? toks * heads : a.queries;
  const size_t first_row = static_cast<size_t>(u) * a.queries + tok0 * heads;
  const int n_old = a.n_used[u];
  const int n = min(B, n_old + a.block);
  const int qp0 = a.qpos0[u];
  const bool evicted = n_old >= B;
  int fresh = -1;
  if (SINGLE) {
    fresh = evicted ? min(a.next_slot[u], B - 1) : n_old;
    if (HD == 64 && fresh < 0)  // (bf16 / 128 takes slot 0)
      fresh = victim_by_statistics<NT, PER_WORD>(a.stats + static_cast<size_t>(u) * 3 * B, a.pos + static_cast<size_t>(u) * B, B, a.pol, a.scope,
                                                 sel_sh, best_sh);
    fresh = max(fresh, 0);
  }
  char* const Kb = static_cast<char*>(a.K) + static_cast<size_t>(u) * B * kRowBytes;
  char* const Vb = static_cast<char*>(a.V) + static_cast<size_t>(u) * B * kRowBytes;
  int32_t* const pos = a.pos + static_cast<size_t>(u) * B;

  // ---- the stream: wave w takes every W-th tile of 32 slots, K first, from a start that differs between workgroups; stage t % 2
  const v4i32 kbuf = make_buffer(Kb, static_cast<uint32_t>(n) * kRowBytes);  // rows behind the last slot come back as zeros
  const v4i32 vbuf = make_buffer(Vb, static_cast<uint32_t>(n) * kRowBytes);
  const v4i32 pbuf = make_buffer(pos, static_cast<uint32_t>(B) * 4u);
  char* const tiles = lds + wave * kTileBytes;  // stage s: W tiles further
  const uint32_t tiles_addr = lds_address(tiles), pos_addr = lds_address(&pos_s[WINDOW ? wave : 0][0][0]);
  // (the scalar offset of a request is the tile's first row, which exists: see load16_to_lds)
  const int n_tiles = (n + kTileSlots - 1) / kTileSlots;
  const int mine = (n_tiles - wave + W - 1) / W;
  const int rot = mine > 0 ? static_cast<int>((static_cast<unsigned>(u) * 5u) % static_cast<unsigned>(mine)) : 0;
  auto tile_of = [&](int t) { return t + rot < mine ? t + rot : t + rot - mine; };  // index among the wave's tiles
  auto tile_row = [&](int t) { return (tile_of(t) * W + wave) * kTileSlots; };
  const int load_row = lane / R::kChunks, load_slot = lane % R::kChunks;  // of a wave-wide load
  auto request_k = [&](int t) {
    const int row = tile_row(t);
    const int soff = __builtin_amdgcn_readfirstlane(row * kRowBytes);
    const uint32_t dst = tiles_addr + (t & 1) * (W * kTileBytes);
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
      const int r = R::kPerLoad * i + load_row;
      load16_to_lds_hint<STREAMING>(kbuf, dst + i * 1024, r * kRowBytes + ((load_slot ^ R::swizzle_k(r)) << 4), soff);
    }
    if (WINDOW) load4_to_lds(pbuf, pos_addr + (t & 1) * (kWave * 4), lane * 4, __builtin_amdgcn_readfirstlane(row * 4));
  };
  auto request_v = [&](int t) {
    const int soff = __builtin_amdgcn_readfirstlane(tile_row(t) * kRowBytes);
    const uint32_t dst = tiles_addr + (t & 1) * (W * kTileBytes);
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
      const int r = R::kPerLoad * i + load_row;
      load16_to_lds_hint<STREAMING>(vbuf, dst + i * 1024, r * kRowBytes + ((load_slot ^ R::swizzle_v(r)) << 4), soff);
    }
  };
  const bool mine_first = !TURNS || (u & 8) == 0;  // neighbours on a die take turns (see above)
  const bool evict_first = !SINGLE && mine_first, v_first = !mine_first;
  const bool v_ahead = v_room && !v_first;
  if (mine > 0 && !evict_first) request_k(0);

  // B operand: the queries (lanes beyond the step's repeat its last one; their results are dropped)
  uint4 own[NQ][R::kSteps];
#pragma unroll
  for (int t2 = 0; t2 < NQ; ++t2) {
    const char* qrow = static_cast<const char*>(a.q) + (first_row + min(kQ16 * t2 + qi, nq - 1)) * kRowBytes;
#pragma unroll
    for (int kk = 0; kk < R::kSteps; ++kk) own[t2][kk] = load16(qrow + kk * 64 + g * 16);
  }
  const float sc = a.scale_log2, rb = a.recency_bias_log2;
  const int w = a.recency_window;
  int qp[NQ];  // this lane's position per query tile; the heads of a group share it
#pragma unroll
  for (int t2 = 0; t2 < NQ; ++t2) qp[t2] = qp0 + (SINGLE ? 0 : tok0 + (kQ16 * t2 + qi) / heads);
  auto logit = [&](float score, int t2, int p) {
    float x = score * sc;
    if (WINDOW) {
      const int dlt = qp[t2] - p;
      if (dlt >= 0 && dlt < w) x += rb;
    }
    return x;
  };
  // The logits of the block's own tokens come from k_new: the slots' rows may have been requested before they were written.
  if (!SINGLE && wave == 0) {
#pragma unroll 1
    for (int t0 = 0; t0 < a.block; t0 += kQ16) {
      const char* krow = static_cast<const char*>(a.k_new) + (static_cast<size_t>(u) * a.block + min(t0 + qi, a.block - 1)) * kRowBytes;
      uint4 kn[R::kSteps];
#pragma unroll
      for (int kk = 0; kk < R::kSteps; ++kk) kn[kk] = load16(krow + kk * 64 + g * 16);
#pragma unroll
      for (int t2 = 0; t2 < NQ; ++t2) {
        f32x4 s = f32x4{0};
#pragma unroll
        for (int kk = 0; kk < R::kSteps; ++kk) s = mfma16(kn[kk], own[t2][kk], s);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int tok = t0 + 4 * g + e;  // a query does not see later tokens of the block
          if (tok < a.block) new_s[kQ16 * t2 + qi][tok] = qp0 + tok > qp[t2] ? -INFINITY : logit(s[e], t2, qp0 + tok);
        }
      }
    }
  }
  // ---- the eviction, before or behind the scores; its keys lie in the second stage
  auto evict = [&]() {
    uint32_t* const keys = reinterpret_cast<uint32_t*>(lds + W * kTileBytes);
    take_slots<NT, PER_WORD, !HALVES>(a, u, n_old, keys, keys + B, sel_sh, scan_sh, slot_of, [&](int j, int bi) {
      bidx_s[j] = static_cast<signed char>(bi);
      if (HALVES && tok0 == 0) a.blk_idx[static_cast<size_t>(u) * B + j] = bi;
    });
    __syncthreads();  // the keys have been used, the block's rows are in the cache
  };
  if (evict_first) evict();
  // A single token's row, put over what its slot held, in the tile if it is there and in the cache: 16 lanes.
  auto put_row = [&](const void* rows, char* cache, char* tile, int slot_in_tile, int swizzle) {
    if (static_cast<unsigned>(slot_in_tile) < static_cast<unsigned>(kTileSlots) && lane < R::kChunks) {
      const uint4 row = load16(static_cast<const char*>(rows) + static_cast<size_t>(u) * kRowBytes + lane * 16);
      *reinterpret_cast<uint4*>(tile + slot_in_tile * kRowBytes + ((lane ^ swizzle) << 4)) = row;
      *reinterpret_cast<uint4*>(cache + static_cast<size_t>(fresh) * kRowBytes + lane * 16) = row;
    }
  };
  f32x4 z[ZT][NQ][2];  // logits, then probabilities
#pragma unroll
  for (int i = 0; i < ZT; ++i)
#pragma unroll
    for (int t2 = 0; t2 < NQ; ++t2) z[i][t2][0] = z[i][t2][1] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};

  {
    // ---- scores
    if (mine > 0 && evict_first) request_k(0);
    if (mine > 1) request_k(1);
    const int kfrag = qi * kRowBytes + ((g ^ R::swizzle_k(qi)) << 4);
#pragma unroll 1
    for (int t = 0; t < mine; ++t) {
      const int sb = tile_row(t);
      const int zt = tile_of(t);
      char* const tile = tiles + (t & 1) * (W * kTileBytes);
      if (t + 1 < mine) wait_loads<kTileLoads + kSide>();
      else wait_loads<0>();
      if (SINGLE) put_row(a.k_new, Kb, tile, fresh - sb, R::swizzle_k(fresh - sb));
      f32x4 s[NQ][2];
#pragma unroll
      for (int kk = 0; kk < R::kSteps; ++kk) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint4 kf = *reinterpret_cast<const uint4*>(tile + h * 16 * kRowBytes + (kfrag ^ (kk << 6)));
#pragma unroll
          for (int t2 = 0; t2 < NQ; ++t2) s[t2][h] = mfma16(kf, own[t2][kk], kk == 0 ? f32x4{0} : s[t2][h]);
        }
      }
      int ps[2][4];
      if (WINDOW) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int4 p4 = *reinterpret_cast<const int4*>(&pos_s[WINDOW ? wave : 0][t & 1][16 * h + 4 * g]);
          ps[h][0] = p4.x; ps[h][1] = p4.y; ps[h][2] = p4.z; ps[h][3] = p4.w;
        }
      }
      reads_done();
      if (t + 2 < mine) request_k(t + 2);
#pragma unroll
      for (int t2 = 0; t2 < NQ; ++t2)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int slot = sb + 16 * h + 4 * g + e;
            const float x = logit(s[t2][h][e], t2, !WINDOW ? 0 : SINGLE && slot == fresh ? qp0 : ps[h][e]);
            s[t2][h][e] = slot < n ? x : -INFINITY;
          }
#pragma unroll
      for (int i = 0; i < ZT; ++i) {
        if (zt == i) {
#pragma unroll
          for (int t2 = 0; t2 < NQ; ++t2)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              z[i][t2][h] = s[t2][h];
              asm volatile("" : "+v"(z[i][t2][h]));  // (kept a branch: as selects it is a move per register and tile)
            }
        }
      }
    }
  }
  __syncthreads();  // nobody needs the tiles of K any more, and new_s has been written
  if (!SINGLE && TURNS && !evict_first) evict();

  // the statistics of the thread's slots, four in a row of every lds_slots, and the first tile of V are requested now
  float* const acc = a.stats + static_cast<size_t>(u) * 3 * B;
  float* const acc2 = acc + B;
  float* const cnt = acc2 + B;
  float4 a1, a2, cc;
  auto load_stats = [&](int c0) {
    const int j = tid * 4 < lds_slots && c0 + tid * 4 < n ? c0 + tid * 4 : 0;
    a1 = *reinterpret_cast<const float4*>(acc + j);
    a2 = *reinterpret_cast<const float4*>(acc2 + j);
    cc = *reinterpret_cast<const float4*>(cnt + j);
  };
  if (!HALVES) load_stats(0);
  if (v_ahead && mine > 0) request_v(0);

  // ---- the block's own tokens take the place of what the slots held
#pragma unroll 1
  for (int tok = 0; !SINGLE && tok < a.block; ++tok) {
    const int slot = __builtin_amdgcn_readfirstlane(slot_of[tok]);
    const int tile = slot / kTileSlots;
    if (tile % W != wave) continue;
    const int zt = tile / W, h1 = (slot >> 4) & 1, e1 = slot & 3;
    const bool my_slots = g == ((slot >> 2) & 3);
    float x[NQ];
#pragma unroll
    for (int t2 = 0; t2 < NQ; ++t2) x[t2] = new_s[kQ16 * t2 + qi][tok];
#pragma unroll
    for (int i = 0; i < ZT; ++i) {
      if (zt == i) {
#pragma unroll
        for (int t2 = 0; t2 < NQ; ++t2)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (h == h1 && e == e1) z[i][t2][h][e] = my_slots ? x[t2] : z[i][t2][h][e];
            asm volatile("" : "+v"(z[i][t2][h]));
          }
      }
    }
  }

  // ---- normalisers
  float M[NQ];
#pragma unroll
  for (int t2 = 0; t2 < NQ; ++t2) {
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < ZT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) m = max3(max3(m, z[i][t2][h][0], z[i][t2][h][1]), z[i][t2][h][2], z[i][t2][h][3]);
    m = fmaxf(m, __shfl_xor(m, 16, kWave));
    m = fmaxf(m, __shfl_xor(m, 32, kWave));
    if (g == 0) m_s[wave][kQ16 * t2 + qi] = m;
  }
  __syncthreads();
#pragma unroll
  for (int t2 = 0; t2 < NQ; ++t2) {
    M[t2] = -INFINITY;
#pragma unroll
    for (int i = 0; i < W; ++i) M[t2] = fmaxf(M[t2], m_s[i][kQ16 * t2 + qi]);
    float l = 0.0f;
#pragma unroll
    for (int i = 0; i < ZT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z[i][t2][h][e] = fast_exp2(z[i][t2][h][e] - M[t2]);
          l += z[i][t2][h][e];
        }
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    if (g == 0) l_s[wave][kQ16 * t2 + qi] = l;
  }
  __syncthreads();
  bool odd = false;  // one of the lane's rows is NaN
#pragma unroll
  for (int t2 = 0; t2 < NQ; ++t2) {
    float L = 0.0f;
#pragma unroll
    for (int i = 0; i < W; ++i) L += l_s[i][kQ16 * t2 + qi];
    odd = odd || !(L < INFINITY);
    const float inv = 1.0f / L;
#pragma unroll
    for (int i = 0; i < ZT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) z[i][t2][h] *= inv;
  }

  const bool odd_rows = !SINGLE && __builtin_amdgcn_ballot_w64(odd) != 0;  // (every wave has all rows)

  auto statistics = [&]() {
    // ---- statistics: every slot receives, per block token that attended it, the head-mean of the probabilities
    const float inv_heads = 1.0f / static_cast<float>(heads);
    const bool full = n >= B;
    const bool squares = !a.pol.keeps_last_score() && !a.pol.counts_above_average();
    uint32_t* const var_key = reinterpret_cast<uint32_t*>(lds + (v_ahead ? W * kTileBytes : 0));  // [B], behind it mas_key, then the probabilities of lds_slots slots
    uint32_t* const mas_key = var_key + B;
    float* const pl = reinterpret_cast<float*>(mas_key + B);
    const int prow = lds_slots + 4;
    const int chunk_tiles = lds_slots / (W * kTileSlots);
#pragma unroll 1
    for (int c0 = 0; c0 < n; c0 += lds_slots) {
      const int i0 = c0 / (W * kTileSlots);
      if (c0 > 0) __syncthreads();  // the slots before have been dealt with
#pragma unroll
      for (int i = 0; i < ZT; ++i) {
        if (i >= i0 && i < i0 + chunk_tiles) {
          const int slot0 = ((i - i0) * W + wave) * kTileSlots + 4 * g;
#pragma unroll
          for (int t2 = 0; t2 < NQ; ++t2) {
            const int q = kQ16 * t2 + qi;
            if (q < nq) {
#pragma unroll
              for (int h = 0; h < 2; ++h) *reinterpret_cast<f32x4*>(pl + static_cast<size_t>(q) * prow + slot0 + 16 * h) = z[i][t2][h];
            }
          }
        }
      }
      __syncthreads();
      if (odd_rows) {  // what a row of NaN did not attend is not NaN (asked here, not at every addition: 512 x 16 tokens x 2048 112 us, 109 so)
#pragma unroll 1
        for (int i = tid; i < nq * a.block; i += NT) {
          const int q = i / a.block, tok = i % a.block, slot = slot_of[tok] - c0;
          if (tok > tok0 + q / heads && static_cast<unsigned>(slot) < static_cast<unsigned>(lds_slots)) pl[static_cast<size_t>(q) * prow + slot] = 0.0f;
        }
        __syncthreads();
      }
      const int j = c0 + tid * 4;
      const float4 b1 = a1, b2 = a2, bc = cc;
      if (!HALVES) load_stats(c0 + lds_slots);
      if (tid * 4 < lds_slots && j < n) {
        float s1[4] = {b1.x, b1.y, b1.z, b1.w}, s2[4] = {b2.x, b2.y, b2.z, b2.w}, sc4[4] = {bc.x, bc.y, bc.z, bc.w};
        if (HALVES) {
#pragma unroll
          for (int e = 0; e < 4; ++e) s1[e] = s2[e] = 0.0f;
        }
        int bi[4] = {-1, -1, -1, -1};
        if (!SINGLE) {
          const int b4 = *reinterpret_cast<const int*>(bidx_s + j);
#pragma unroll
          for (int e = 0; e < 4; ++e) bi[e] = (b4 << (24 - 8 * e)) >> 24;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (SINGLE ? j + e == fresh : bi[e] >= 0) { s1[e] = 0.0f; s2[e] = 0.0f; sc4[e] = 0.0f; }  // a new token starts from zero
        const float* prob = pl + tid * 4;
        // A token that did not attend a slot (it is older than the one that the slot holds) gave it a probability of zero.
        auto add = [&](int t, const float4& mean) {
          const float p[4] = {mean.x * inv_heads, mean.y * inv_heads, mean.z * inv_heads, mean.w * inv_heads};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s1[e] += p[e];
            if (HALVES || squares) s2[e] += p[e] * p[e];
            else if (bi[e] <= t) s2[e] = a.pol.second_statistic(s2[e], p[e], static_cast<float>(n - a.block + t + 1));
          }
        };
        if (!SINGLE && heads == 1) {
#pragma unroll 1
          for (int t = 0; t < nq; t += 4) {
            float4 zz[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) zz[i] = *reinterpret_cast<const float4*>(prob + static_cast<size_t>(min(t + i, nq - 1)) * prow);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (t + i < nq) add(t + i, zz[i]);
          }
        } else {
#pragma unroll 1
          for (int t = 0; t < toks; ++t) {
            float4 mean = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 4
            for (int h = 0; h < heads; ++h, prob += prow) {
              const float4 zz = *reinterpret_cast<const float4*>(prob);
              mean.x += zz.x; mean.y += zz.y; mean.z += zz.z; mean.w += zz.w;
            }
            add(t, mean);
          }
        }
        if (HALVES) {  // block_book adds both halves' sums
          float* const part = part_sums(a, u, tok0 != 0);
          *reinterpret_cast<float4*>(part + j) = make_float4(s1[0], s1[1], s1[2], s1[3]);
          *reinterpret_cast<float4*>(part + B + j) = make_float4(s2[0], s2[1], s2[2], s2[3]);
          continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (j + e < n) sc4[e] += static_cast<float>(a.block - max(bi[e], 0));
        }
        if (j + 3 >= n) {  // slots that do not exist keep what they hold
          if (j + 1 >= n) { s1[1] = b1.y; s2[1] = b2.y; }
          if (j + 2 >= n) { s1[2] = b1.z; s2[2] = b2.z; }
          if (j + 3 >= n) { s1[3] = b1.w; s2[3] = b2.w; }
        }
        *reinterpret_cast<float4*>(acc + j) = make_float4(s1[0], s1[1], s1[2], s1[3]);
        *reinterpret_cast<float4*>(acc2 + j) = make_float4(s2[0], s2[1], s2[2], s2[3]);
        *reinterpret_cast<float4*>(cnt + j) = make_float4(sc4[0], sc4[1], sc4[2], sc4[3]);
        if (full) {  // then all four are slots of the unit
          int pv[4] = {0, 0, 0, 0};
          if (a.pol.needs_pos()) {
#pragma unroll
            for (int e = 0; e < 4; ++e) pv[e] = SINGLE && j + e == fresh ? qp0 : pos[j + e];
          }
          uint4 mk, vk;
          ranking_keys<4>(s1, s2, sc4, pv, a.pol, &mk.x, &vk.x);
          *reinterpret_cast<uint4*>(mas_key + j) = mk;
          *reinterpret_cast<uint4*>(var_key + j) = vk;
        }
      }
    }
    // the victim a following single-token step would take
    int victim = -1;
    if (!HALVES && full) {
      __syncthreads();
      victim = select_victim_block<NT, PER_WORD>(var_key, mas_key, B, a.pol, a.scope, sel_sh, best_sh);
    }
    if (!HALVES && tid == 0) {
      a.next_slot[u] = victim;
      a.n_used[u] = n;
      if (SINGLE) {
        const int old_pos = pos[fresh];
        pos[fresh] = qp0;
        if (a.evicted_slot) a.evicted_slot[u] = evicted ? fresh : -1;
        if (a.evicted_pos) a.evicted_pos[u] = evicted ? old_pos : -1;
      }
    }
    __syncthreads();  // nobody needs the keys and probabilities any more
  };

  auto outputs = [&]() {
    // ---- O^T = V^T . P^T
    if (!v_ahead && mine > 0) request_v(0);
    if (mine > 1) request_v(1);
    f32x4 o[NQ][R::kBlocks];
#pragma unroll
    for (int t2 = 0; t2 < NQ; ++t2)
#pragma unroll
      for (int db = 0; db < R::kBlocks; ++db) o[t2][db] = f32x4{0};
    // V^T of dimensions 0..15: rows 4 g + lane / 4 % 4 of either half of the tile, 8 bytes from column 4 (lane % 4) on
    const int vrow = 4 * g + (qi >> 2);
    const int vfrag = vrow * kRowBytes + (R::swizzle_v(vrow) << 4) + (qi & 3) * 8;
#pragma unroll 1
    for (int t = 0; t < mine; ++t) {
      const int zt = tile_of(t), sb = tile_row(t);
      char* const tile = tiles + (t & 1) * (W * kTileBytes);
      f32x4 x[NQ][2];
#pragma unroll
      for (int i = 0; i < ZT; ++i) {
        if (zt == i) {
#pragma unroll
          for (int t2 = 0; t2 < NQ; ++t2) {
            x[t2][0] = z[i][t2][0];
            x[t2][1] = z[i][t2][1];
            asm volatile("" : "+v"(x[t2][0]), "+v"(x[t2][1]));  // (kept a branch, as above)
          }
        }
      }
      uint4 p[NQ][R::kPlanes];
#pragma unroll
      for (int t2 = 0; t2 < NQ; ++t2) split_positive(x[t2], p[t2]);
      if (t + 1 < mine) wait_loads<kTileLoads>();
      else wait_loads<0>();
      if (SINGLE) put_row(a.v_new, Vb, tile, fresh - sb, R::swizzle_v(fresh - sb));
#pragma unroll
      for (int db = 0; db < R::kBlocks; ++db) {
        const char* const vt = tile + (vfrag ^ (db << 5));
        const uint2 lo = lds_read_transposed(vt), hi = lds_read_transposed(vt + 16 * kRowBytes);
        const uint4 vf = make_uint4(lo.x, lo.y, hi.x, hi.y);
#pragma unroll
        for (int i = R::kPlanes - 1; i >= 0; --i)
#pragma unroll
          for (int t2 = 0; t2 < NQ; ++t2) o[t2][db] = mfma16(vf, p[t2][i], o[t2][db]);
      }
      reads_done();
      if (t + 2 < mine) request_v(t + 2);
    }
    __syncthreads();  // nobody needs the tiles any more
    float* const outs = reinterpret_cast<float*>(lds);  // [W][QR][R::kOut]
#pragma unroll
    for (int t2 = 0; t2 < NQ; ++t2) {
      const int q = kQ16 * t2 + qi;
      if (q < nq) {
#pragma unroll
        for (int db = 0; db < R::kBlocks; ++db) *reinterpret_cast<f32x4*>(outs + (wave * QR + q) * R::kOut + 16 * db + 4 * g) = o[t2][db];
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int idx = tid * 4; idx < nq * HD; idx += NT * 4) {
      const int q = idx / HD, dd = idx % HD;
      f32x4 sum = f32x4{0};
#pragma unroll
      for (int i = 0; i < W; ++i) sum += *reinterpret_cast<const f32x4*>(outs + (i * QR + q) * R::kOut + dd);
      uint2 r;
      r.x = f32_to_bf16(sum.x) | static_cast<uint32_t>(f32_to_bf16(sum.y)) << 16;
      r.y = f32_to_bf16(sum.z) | static_cast<uint32_t>(f32_to_bf16(sum.w)) << 16;
      *reinterpret_cast<uint2*>(static_cast<char*>(a.out) + (first_row * HD + idx) * 2) = r;
    }
  };

  if constexpr (!TURNS) {
    statistics();
    outputs();
  } else {
#pragma unroll 1
    for (int phase = 0; phase < 2; ++phase) {
      if ((phase == 0) != v_first) {
        statistics();
      } else {
        outputs();
        __syncthreads();  // nobody needs the outputs any more
      }
    }
  }
}

// Behind the two halves of a step: adds their sums to the statistics, books the tokens' slots and chooses the next victim.
constexpr int kBookThreads = 512;
template <int NT>
__global__ __launch_bounds__(NT, 2) void block_book(BlockArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // [2][B] ranking keys
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<1>::kWords];
  __shared__ uint2 best_sh[NT / kWave];
  const int u = blockIdx.x, tid = threadIdx.x, B = a.B;
  const int n_old = a.n_used[u], n = min(B, n_old + a.block), qp0 = a.qpos0[u];
  float* const acc = a.stats + static_cast<size_t>(u) * 3 * B;
  const float *const p0 = part_sums(a, u, 0), *const p1 = part_sums(a, u, 1);
  uint32_t* const var_key = reinterpret_cast<uint32_t*>(lds);
  uint32_t* const mas_key = var_key + B;
  const bool full = n >= B;
#pragma unroll 1
  for (int j = tid * 4; j < n; j += NT * 4) {
    auto at = [&](const float* plane) { return *reinterpret_cast<const f32x4*>(plane + j); };
    const f32x4 o1 = at(acc), o2 = at(acc + B), oc = at(acc + 2 * B);
    float s1[4] = {o1.x, o1.y, o1.z, o1.w}, s2[4] = {o2.x, o2.y, o2.z, o2.w}, sc[4] = {oc.x, oc.y, oc.z, oc.w};
    const f32x4 a1 = at(p0) + at(p1), a2 = at(p0 + B) + at(p1 + B);
    const int4 b4 = *reinterpret_cast<const int4*>(a.blk_idx + static_cast<size_t>(u) * B + j);
    const int4 p4 = *reinterpret_cast<const int4*>(a.pos + static_cast<size_t>(u) * B + j);
    const int bi[4] = {b4.x, b4.y, b4.z, b4.w};
    int pv[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (j + e >= n) continue;  // slots that do not exist keep what they hold
      const bool fresh = bi[e] >= 0;
      s1[e] = (fresh ? 0.0f : s1[e]) + a1[e];
      s2[e] = (fresh ? 0.0f : s2[e]) + a2[e];
      sc[e] = (fresh ? 0.0f : sc[e]) + static_cast<float>(a.block - max(bi[e], 0));  // older tokens were attended by all
      if (fresh) {
        book_slot(a, u, n_old, j + e, bi[e]);
        pv[e] = qp0 + bi[e];
      }
    }
    *reinterpret_cast<float4*>(acc + j) = make_float4(s1[0], s1[1], s1[2], s1[3]);
    *reinterpret_cast<float4*>(acc + B + j) = make_float4(s2[0], s2[1], s2[2], s2[3]);
    *reinterpret_cast<float4*>(acc + 2 * B + j) = make_float4(sc[0], sc[1], sc[2], sc[3]);
    if (full) {  // then all four are slots of the unit
      uint4 mk, vk;
      ranking_keys<4>(s1, s2, sc, pv, a.pol, &mk.x, &vk.x);
      *reinterpret_cast<uint4*>(mas_key + j) = mk;
      *reinterpret_cast<uint4*>(var_key + j) = vk;
    }
  }
  int victim = -1;
  __syncthreads();  // every thread has read n_used
  if (full) victim = select_victim_block<NT, 1>(var_key, mas_key, B, a.pol, a.scope, sel_sh, best_sh);
  if (tid == 0) {
    a.next_slot[u] = victim;
    a.n_used[u] = n;
  }
}

constexpr size_t kLdsOfUnit = 160 << 10;  // of a compute unit

template <int HD, int W, int NQ, int ZT> struct Shape {
  static constexpr int kStep = kTileSlots * W;
  static size_t bytes_of(const BlockArgs& a, int slots) { return (2 * static_cast<size_t>(a.B) + static_cast<size_t>(a.queries) * (slots + 4)) * 4; }
  // what block_fused declares statically, at most
  static constexpr size_t fixed(bool single, bool window, bool halves) {
    const size_t qr = NQ * kQ16;
    const size_t own = single ? qr * 4 + 16 : qr * (halves ? kMaxBlock : qr) * 4 + kStep * ZT;
    return SelectLds<W == 4 ? 2 : 1>::kWords * 4 + (window ? W * 512 : 512) + 2 * W * qr * 4 + qr * 4 + own + 1024;
  }
  // The dynamic LDS of any step, the limit that every launch of a kernel sets: one that followed the step could be lowered by another
  // thread's before the launch.  (Four waves: two workgroups share a compute unit.)
  static constexpr size_t most(bool single, bool window, bool halves) { return kLdsOfUnit / (8 / W) - fixed(single, window, halves); }
  static size_t most(const BlockArgs& a) { return most(a.single != 0, a.recency_window > 0, a.queries < a.block * a.heads); }
  // slots whose probabilities the LDS takes at a time beside the unit's ranking keys, and `ahead` bytes of V; 0: none
  static int slots(const BlockArgs& a, size_t ahead) {
    const size_t room = most(a) - ahead;
    int s = std::min((a.B + kStep - 1) / kStep * kStep, 4 * W * kWave);
    while (s > 0 && bytes_of(a, s) > room) s -= kStep;
    return s;
  }
  static constexpr size_t kStage = W * Rows<HD>::kTile;
  // whether the first tiles of V may be on their way meanwhile
  static bool v_ahead(const BlockArgs& a) { return W == 8 && slots(a, kStage) >= std::min(a.B, 4 * W * kWave); }
  static constexpr size_t kOuts = static_cast<size_t>(W) * NQ * kQ16 * Rows<HD>::kOut * sizeof(float);
  static_assert(std::max(2 * kStage, kOuts) <= std::min(most(false, true, W == 8), most(true, true, false)), "tiles and outputs fit");
  static size_t lds(const BlockArgs& a) {
    const size_t ahead = v_ahead(a) ? kStage : 0;
    return std::max({2 * kStage, kOuts, ahead + bytes_of(a, slots(a, ahead))});
  }
  static bool takes(const BlockArgs& a) { return a.B <= kStep * ZT && a.queries <= kQ16 * NQ && slots(a, 0) > 0; }
};

// The larger half of a step's tokens, as a step of its own.
inline BlockArgs half_step(BlockArgs a) {
  a.queries = (a.block + 1) / 2 * a.heads;
  return a;
}

template <int HD, int W, int NQ, int ZT, bool SINGLE, bool STREAMING, bool WINDOW>
hipError_t launch_t(const BlockArgs& a, hipStream_t s) {
  using S = Shape<HD, W, NQ, ZT>;
  const size_t lds = S::lds(a);
  const void* fn = reinterpret_cast<const void*>(block_fused<HD, W, NQ, ZT, SINGLE, STREAMING, WINDOW>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(S::most(SINGLE, WINDOW, false))) != hipSuccess)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((block_fused<HD, W, NQ, ZT, SINGLE, STREAMING, WINDOW>), dim3(a.units), dim3(W * kWave), lds, s, a,
                     S::slots(a, S::v_ahead(a) ? S::kStage : 0), S::v_ahead(a) ? 1 : 0);
  return hipSuccess;
}
template <int HD, int W, int NQ, int ZT>
hipError_t launch(const BlockArgs& a, hipStream_t s) {
  const bool window = a.recency_window > 0;
  if (a.single) {
    if (a.streaming) return window ? launch_t<HD, W, NQ, ZT, true, true, true>(a, s) : launch_t<HD, W, NQ, ZT, true, true, false>(a, s);
    return window ? launch_t<HD, W, NQ, ZT, true, false, true>(a, s) : launch_t<HD, W, NQ, ZT, true, false, false>(a, s);
  }
  if (a.streaming) return window ? launch_t<HD, W, NQ, ZT, false, true, true>(a, s) : launch_t<HD, W, NQ, ZT, false, true, false>(a, s);
  return window ? launch_t<HD, W, NQ, ZT, false, false, true>(a, s) : launch_t<HD, W, NQ, ZT, false, false, false>(a, s);
}

template <int HD, int W, int NQ, int ZT, bool STREAMING, bool WINDOW>
hipError_t launch_halves_t(const BlockArgs& a, const BlockArgs& half, hipStream_t s) {
  using S = Shape<HD, W, NQ, ZT>;
  const size_t lds = S::lds(half);
  const void* fn = reinterpret_cast<const void*>(block_fused<HD, W, NQ, ZT, false, STREAMING, WINDOW, true>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(S::most(false, WINDOW, true))) != hipSuccess)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((block_fused<HD, W, NQ, ZT, false, STREAMING, WINDOW, true>), dim3((a.units + 7) / 8 * 16), dim3(W * kWave), lds, s, a,
                     S::slots(half, S::v_ahead(half) ? S::kStage : 0), S::v_ahead(half) ? 1 : 0);
  hipLaunchKernelGGL((block_book<kBookThreads>), dim3(a.units), dim3(kBookThreads), key_lds_bytes(a.B), s, a);
  return hipSuccess;
}
template <int HD, int W, int NQ, int ZT>
hipError_t launch_halves(const BlockArgs& a, hipStream_t s) {
  const BlockArgs half = half_step(a);
  const bool window = a.recency_window > 0;
  if (a.streaming) return window ? launch_halves_t<HD, W, NQ, ZT, true, true>(a, half, s) : launch_halves_t<HD, W, NQ, ZT, true, false>(a, half, s);
  return window ? launch_halves_t<HD, W, NQ, ZT, false, true>(a, half, s) : launch_halves_t<HD, W, NQ, ZT, false, false>(a, half, s);
}

}  // namespace fused
}  // namespace roco
