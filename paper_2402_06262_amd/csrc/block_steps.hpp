// What the kernels of the block-wise step share: the choice of the victims, the order in which the block's tokens take the freed and
// the still-empty slots, and the loads that take a wave's tiles straight to LDS.
#pragma once
#include "kernels.hpp"
#include "mfma.hpp"
#include "stream.hpp"
#include "tile_ring.hpp"

namespace roco {

// Slot j of a unit that held n tokens takes block token bi: pos, and the record of what was evicted.
__device__ __forceinline__ void book_slot(const BlockArgs& a, int u, int n, int j, int bi) {
  int32_t* const pos = a.pos + static_cast<size_t>(u) * a.B;
  const bool held = j < n;  // the slot held a token that is now evicted
  if (a.evicted_slot) a.evicted_slot[static_cast<size_t>(u) * a.block + bi] = held ? j : -1;
  if (a.evicted_pos) a.evicted_pos[static_cast<size_t>(u) * a.block + bi] = held ? pos[j] : -1;
  pos[j] = a.qpos0[u] + bi;
}

// The step's E = max(0, n + b - B) victims (two exact searches), the slots its tokens take, their K / V rows in the cache and, with
// BOOK, book_slot.  place(j, bi) says of every slot which block token it now holds (-1: an older one, or none).
// The ranking keys lie in var_key[B] and mas_key[B].  The two selections share one copy of the search: a launch starts with a cold
// instruction cache.  Ends with a barrier behind the last write of slot_of, not behind the rows.
template <int NT, int PER_WORD, bool BOOK, class Place>
__device__ __forceinline__ void take_slots(const BlockArgs& a, int u, int n, uint32_t* var_key, uint32_t* mas_key, uint32_t* sel_sh,
                                           uint32_t* scan_sh, int* slot_of, Place place) {
  const int tid = threadIdx.x;
  const int B = a.B, b = a.block;
  const int E = max(0, n + b - B);
  const int n_new = min(B, n + b);
  const float* acc = a.stats + static_cast<size_t>(u) * 3 * B;
  const float* acc2 = acc + B;
  const float* cnt = acc2 + B;
  const int32_t* pos = a.pos + static_cast<size_t>(u) * B;

  // The block's K / V rows (16 bytes per lane, a power of two of lanes per row) are requested now and stored at the end: the
  // first NT / lanes rows are under way while the victims are chosen (16 tokens on 512 units: 23.4 -> 21.5 us).
  const int lanes_log2 = __builtin_ctz(a.row_bytes) - 4;
  const int my_row = tid >> lanes_log2, my_col = (tid & ((1 << lanes_log2) - 1)) * 16;
  const size_t in_base = static_cast<size_t>(u) * b * a.row_bytes + my_col;
  auto new_row = [&](const void* rows, int i) { return load16(static_cast<const char*>(rows) + in_base + static_cast<size_t>(i) * a.row_bytes); };
  const int safe_row = min(my_row, b - 1);
  uint4 k_row = new_row(a.k_new, safe_row), v_row = new_row(a.v_new, safe_row);

  if (tid < kMaxBlock) slot_of[tid] = 0;
  KSmallest scope = {0u, 0u}, out = {0u, 0u};
  // one eviction from a full cache: the victim was already chosen when the statistics were last updated
  const int hint = (E == 1 && n == B) ? a.next_slot[u] : -1;
  if (E > 0 && hint < 0) {
    // (B is a multiple of 4 on this path: four slots are inside the planes, and the keys behind the last slot are not read)
#pragma unroll 1
    for (int i = tid * 4; i < n; i += NT * 4) {
      const float4 a1 = *reinterpret_cast<const float4*>(acc + i), a2 = *reinterpret_cast<const float4*>(acc2 + i);
      const float4 cc = *reinterpret_cast<const float4*>(cnt + i);
      const int4 pp = *reinterpret_cast<const int4*>(pos + i);
      uint4 mk, vk;
      ranking_keys<4>(&a1.x, &a2.x, &cc.x, &pp.x, a.pol, &mk.x, &vk.x);
      *reinterpret_cast<uint4*>(mas_key + i) = mk;
      *reinterpret_cast<uint4*>(var_key + i) = vk;
    }
    __syncthreads();
    const uint32_t m = min(static_cast<uint32_t>(n), static_cast<uint32_t>(a.pol.scope_size(a.scope, n)) + static_cast<uint32_t>(E) - 1u);
#pragma unroll 1
    for (int phase = 0; phase < 2; ++phase) {
      const KSmallest r = select_k_smallest<NT, PER_WORD, 1>(
          [&](int i) -> uint32_t {
            const uint32_t vk = var_key[i];
            return phase == 0 ? vk : scope.has(vk, i) ? mas_key[i] : 0xffffffffu;
          },
          n, phase == 0 ? m : static_cast<uint32_t>(E), phase == 0 && a.pol.scope_is_window(), sel_sh, phase == 0 || a.pol.spreads_importance());
      if (phase == 0) scope = r;
      else out = r;
    }
  }
  auto is_target = [&](int j) -> bool {
    if (j >= n) return j < n_new;  // still-empty slot taken by the block
    if (E == 0) return false;
    if (hint >= 0) return j == hint;
    const uint32_t k2 = scope.has(var_key[j], j) ? mas_key[j] : 0xffffffffu;
    return out.has(k2, j);
  };
  // ordered assignment: thread t owns the contiguous slots [t*c, (t+1)*c); the i-th target gets block token i
  const int c = (B + NT - 1) / NT;
  const int lo = min(B, tid * c), hi = min(B, lo + c);
  uint32_t mine = 0;
#pragma unroll 1
  for (int j = lo; j < hi; ++j) mine += (j < n_new && is_target(j)) ? 1u : 0u;
  uint32_t total;
  uint32_t rank = block_exclusive_scan<NT>(mine, scan_sh, total);
#pragma unroll 1
  for (int j = lo; j < hi; ++j) {
    int bi = -1;
    if (j < n_new && is_target(j) && rank < static_cast<uint32_t>(b)) {
      bi = static_cast<int>(rank++);
      slot_of[bi] = j;
      if (BOOK) book_slot(a, u, n, j, bi);
    }
    place(j, bi);
  }
  __syncthreads();
#pragma unroll 1
  for (int i = my_row; i < b;) {
    const size_t dst = (static_cast<size_t>(u) * B + slot_of[i]) * a.row_bytes + my_col;
    *reinterpret_cast<uint4*>(static_cast<char*>(a.K) + dst) = k_row;
    *reinterpret_cast<uint4*>(static_cast<char*>(a.V) + dst) = v_row;
    i += NT >> lanes_log2;
    if (i < b) { k_row = new_row(a.k_new, i); v_row = new_row(a.v_new, i); }
  }
}

// The slot that the token of a single-token step overwrites in a full unit whose next_slot is negative: a cache that its owner has
// put together without roco_select_victims.  By the statistics as they stand, which no kernel has touched yet, as block_prepare
// chooses; the keys are formed as the search reads them, since this is not the path that has to be fast.
template <int NT, int PER_WORD>
__device__ __forceinline__ int victim_by_statistics(const float* stats, const int32_t* pos, int B, Policy pol, int scope, uint32_t* sel_sh,
                                                 uint2* best_sh) {
  auto keys = [&](int i) {
    uint32_t mas_key, var_key;
    ranking_keys(stats[i], stats[B + i], stats[2 * static_cast<size_t>(B) + i], pos[i], pol, mas_key, var_key);
    return make_uint2(mas_key, var_key);
  };
  return select_victim<NT, PER_WORD, false>([&](int i) { return keys(i).y; }, [&](int i) { return keys(i).x; }, B, pol, scope, sel_sh, best_sh);
}

#pragma clang diagnostic ignored "-Winline-asm"
namespace mfma {

template <bool STREAMING>
__device__ __forceinline__ void load16_to_lds_hint(v4i32 rsrc, uint32_t lds_addr, int voffset, int soffset) {
  if (STREAMING)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :: "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset) : "memory", "m0");
  else
    load16_to_lds(rsrc, lds_addr, voffset, soffset);
}
// The wave's LDS reads so far have returned: their tile may be overwritten.
__device__ __forceinline__ void reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace mfma

}  // namespace roco
