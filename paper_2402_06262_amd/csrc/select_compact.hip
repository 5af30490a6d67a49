// Prefill eviction step and cache compaction (one eviction step that frees E = len - B tokens; section 5.3
// "Overhead", block-wise evict-and-encode with the prompt as one block).
//
// Rule (section 4.3 applied E times with the statistics frozen, in closed form): among the s + E - 1
// tokens of lowest attention variance, evict the E tokens of lowest mean attention score; equal keys go to
// the lowest position.  The retained tokens keep ascending position order in the compacted cache.
//
//   prefill_select  : one workgroup per unit.  Two exact k-smallest selections on the fp32 bit patterns
//                     (radix select, no sorting), then an ordered prefix sum assigns cache slots and writes
//                     pos[], the three statistics planes and n_used.
//   prefill_gather  : grid (row blocks, units): copies the retained K / V rows into the cache, 16 bytes per
//                     lane.  Few rows per unit are copied by prefill_select itself.
#include <cstdlib>

#include "kernels.hpp"
#include "profile.hpp"
#include "stream.hpp"

namespace roco {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kGatherThreads = 256;
constexpr int kGatherRows = 64;  // cache rows per gather workgroup

// A launch of this kernel starts with a cold instruction cache and walks through its code once, so the code is kept short:
// the two selections (scope, victims) share one copy of the search, loops over keys in LDS are not
// unrolled, and where the keys are is a template parameter so that they are read with LDS instructions.
// LDS: both keys of a token in LDS (2; up to 16384 tokens), the one of the scope (1; up to 32768), none (0).
// MANY: the column sums lie in more than two shares (LDS = 2).  They are added once, by the thread that will need the sums again
// when it compacts, and left in the first one's planes; for two shares reading both again is faster.
// GATHER: the retained K / V rows are copied here too, by way of the list of their positions in LDS (LDS = 2).  One launch less,
// for units whose rows a compute unit copies in the time that a launch takes: see gathers_in_selection.
template <int LDS, bool MANY, bool GATHER, int NT = kSelThreads>
__global__ __launch_bounds__(NT, 8) void prefill_select(PrefillArgs a) {
  static_assert(LDS == 2 || (!MANY && !GATHER), "the list and the sums replace keys in LDS");
  extern __shared__ __attribute__((aligned(16))) uint32_t lds_keys[];  // [2][L_max] ranking keys when L_max <= kMaxDecodeBudgetLds
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<1>::kWords];
  __shared__ uint32_t scan_sh[NT / kWave + 1];
  __shared__ uint2 best_sh[NT / kWave];
  const int u = blockIdx.x, tid = threadIdx.x;
  const int B = a.B;
  const int n = a.len[u];
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  // the column sums, in one or two shares
  const bool two = LDS == 2 && !MANY && a.shares_to_add == 2;
  float* const first1 = a.acc + ubase;
  float* const first2 = a.acc2 + ubase;
  const float* const second1 = a.sums_of(1, 0) + ubase;
  const float* const second2 = a.sums_of(1, 1) + ubase;
  auto sums = [&](int i) {
    float2 s = make_float2(first1[i], first2[i]);
    if (two) { s.x += second1[i]; s.y += second2[i]; }
    return s;
  };
  if constexpr (MANY) {
#pragma unroll 1
    for (int i = tid; i < n; i += NT) {
      float2 s = make_float2(first1[i], first2[i]);
#pragma unroll 4
      for (int k = 1; k < a.shares_to_add; ++k) { s.x += a.sums_of(k, 0)[ubase + i]; s.y += a.sums_of(k, 1)[ubase + i]; }
      first1[i] = s.x;
      first2[i] = s.y;
    }
  }
  // every radix pass reads every key: in LDS they cost a fraction of a trip to the L2 each
  uint32_t* const var_key = LDS > 0 ? lds_keys : a.var_key + ubase;
  uint32_t* const mas_key = LDS == 2 ? lds_keys + a.L_max : a.mas_key + ubase;
  float* oacc = a.stats + static_cast<size_t>(u) * 3 * B;
  float* oacc2 = oacc + B;
  float* ocnt = oacc2 + B;
  int32_t* pos = a.pos + static_cast<size_t>(u) * B;

  const int kept = n < B ? n : B;
  const uint32_t E = static_cast<uint32_t>(n - kept);
  if (n >= B) {
    auto make_keys = [&](int first, auto tokens) {  // the sums of all tokens are requested before the first is used
      constexpr int N = decltype(tokens)::value;
      float s1[N], s2[N], count[N];
      int p[N];
      uint32_t mk[N], vk[N];
#pragma unroll
      for (int e = 0; e < N; ++e) {
        p[e] = min(first + e * NT, n - 1);
        const float2 s = sums(p[e]);
        s1[e] = s.x; s2[e] = s.y;
        count[e] = static_cast<float>(n - p[e]);
      }
      ranking_keys<N>(s1, s2, count, p, a.pol, mk, vk);
#pragma unroll
      for (int e = 0; e < N; ++e) {
        if (first + e * NT < n) {
          var_key[p[e]] = vk[e];
          mas_key[p[e]] = mk[e];
        }
      }
    };
    if (n <= NT) {
      if (tid < n) make_keys(tid, std::integral_constant<int, 1>{});
    } else {
#pragma unroll 1
      for (int i = tid; i < n; i += 4 * NT) make_keys(i, std::integral_constant<int, 4>{});
    }
    __syncthreads();
  }
  // Phase 0: the scope of the eviction; 1: the victims.  The scope of the first decode step needs no search of its own: the s + E - 1
  // tokens of lowest scope key less the E victims, all of them among these, and the next one, the lowest outside (prompts of 256 /
  // 1000 / 2048 / 4096 tokens: 2.2 / 2.5 / 3.1 / 4.6 us).  Without an eviction phase 0 finds that scope.
  KSmallest scope = {0u, 0u}, out = {0u, 0u};
  if (n >= B) {
#pragma unroll 1
    for (int phase = 0; phase < (E > 0 ? 2 : 1); ++phase) {
      const uint32_t k = phase == 1 ? E
                         : E > 0    ? min(static_cast<uint32_t>(n), static_cast<uint32_t>(a.pol.scope_size(a.scope, n)) + E - 1u)
                                    : static_cast<uint32_t>(a.pol.scope_size(a.scope, B));
      const KSmallest r = select_k_smallest<NT, 1, LDS == 2 ? 1 : 4>(
          [&](int i) -> uint32_t {
            const uint32_t vk = var_key[i];
            if (phase == 0) return vk;
            return scope.has(vk, i) ? mas_key[i] : 0xffffffffu;
          },
          n, k, phase == 0 && a.pol.scope_is_window(), sel_sh, phase == 0 || a.pol.spreads_importance());
      if (phase == 0) scope = r;
      else out = r;
    }
  }
  // ordered compaction, NT positions at a time: a token's slot is the number of retained tokens before it, counted by ballots
  // inside a wave and by the waves' totals in LDS before it
  uint32_t best_key = 0xffffffffu, best = 0xffffffffu, best_slot = 0;  // the least important retained token of the scope
  uint32_t next_key = 0xffffffffu, next = 0xffffffffu, next_slot = 0, next_mas = 0;  // the token of lowest scope key outside
  uint32_t before = 0;  // retained tokens of earlier rounds
  float2 ahead = sums(min(tid, max(n - 1, 0)));  // of the next round: a trip to memory that its barriers hide
#pragma unroll 1
  for (int base = 0; base < n; base += NT) {
    const int i = base + tid;
    const bool in = i < n;
    const float2 s = ahead;
    if (base + NT < n) ahead = sums(min(i + NT, n - 1));
    // (the list of positions grows over keys that have been read: a token's own are read before the barrier)
    const uint32_t vk = in && n >= B ? var_key[i] : 0u, mk = in && n >= B ? mas_key[i] : 0u;
    const bool inside = scope.has(vk, i);
    const bool keep = in && !(E > 0 && out.has(inside ? mk : 0xffffffffu, i));
    const uint64_t votes = __builtin_amdgcn_ballot_w64(keep);
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    __syncthreads();  // the previous round's totals have been read
    if (lane == 0) scan_sh[wave] = __builtin_popcountll(votes);
    __syncthreads();
    const uint32_t totals = wave_inclusive_scan(lane < NT / kWave ? scan_sh[lane] : 0u);
    uint32_t dst = before + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(votes >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(votes), 0));
    if (wave > 0) dst += __builtin_amdgcn_readlane(totals, __builtin_amdgcn_readfirstlane(wave) - 1);
    before += __builtin_amdgcn_readlane(totals, NT / kWave - 1);
    if (keep && dst < static_cast<uint32_t>(B)) {
      pos[dst] = i;
      oacc[dst] = s.x;
      oacc2[dst] = s.y;
      ocnt[dst] = static_cast<float>(n - i);
      if (GATHER) var_key[dst] = static_cast<uint32_t>(i);
      if (inside && (mk < best_key || best == 0xffffffffu)) {
        best_key = mk;
        best = static_cast<uint32_t>(i);
        best_slot = dst;
      }
      if (!inside && (vk < next_key || next == 0xffffffffu)) {
        next_key = vk;
        next = static_cast<uint32_t>(i);
        next_slot = dst;
        next_mas = mk;
      }
    }
  }
#pragma unroll 1
  for (int i = kept + tid; i < B; i += NT) {
    pos[i] = -1;
    oacc[i] = 0.0f;
    oacc2[i] = 0.0f;
    ocnt[i] = 0.0f;
  }
  if (tid == 0) a.n_used[u] = kept;
  // The first decode step on a full cache needs its victim.  (Before the rows are copied: a barrier waits for every store before it,
  // 3 to 4 us where the copies are long.)
  if (kept == B) {
    if (E > 0 && scope.kth != 0xffffffffu) {  // (else the scope is everything)
      const uint32_t last = block_argmin<NT>(next_key, next, best_sh);
      if (last == next && next != 0xffffffffu && (next_mas < best_key || best == 0xffffffffu || (next_mas == best_key && next < best))) {
        best_key = next_mas;
        best = next;
        best_slot = next_slot;
      }
      __syncthreads();  // (best_sh is used again)
    }
    const uint32_t victim = block_argmin<NT>(best_key, best, best_sh);
    if (victim == best) a.next_slot[u] = static_cast<int>(best_slot);  // its owner knows which slot it went to
  } else if (tid == 0) {
    a.next_slot[u] = -1;
  }
  if constexpr (GATHER) {
    __syncthreads();  // the list is whole
    const int lanes_log2 = __builtin_ctz(a.row_bytes) - 4;  // 16 bytes per lane, a power of two of lanes per row
    const int rows = NT >> lanes_log2, col = (tid & ((1 << lanes_log2) - 1)) * 16;
    const char* const Kin = static_cast<const char*>(a.K) + ubase * a.row_bytes + col;
    const char* const Vin = static_cast<const char*>(a.V) + ubase * a.row_bytes + col;
    char* const Kout = static_cast<char*>(a.K_cache) + static_cast<size_t>(u) * B * a.row_bytes + col;
    char* const Vout = static_cast<char*>(a.V_cache) + static_cast<size_t>(u) * B * a.row_bytes + col;
#pragma unroll 1
    for (int slot = tid >> lanes_log2; slot < kept; slot += 2 * rows) {
      const int other = min(slot + rows, kept - 1);  // (copied twice at the end: the same bytes)
      const size_t src0 = static_cast<size_t>(var_key[slot]) * a.row_bytes, src1 = static_cast<size_t>(var_key[other]) * a.row_bytes;
      const uint4 k0 = load16(Kin + src0), v0 = load16(Vin + src0), k1 = load16(Kin + src1), v1 = load16(Vin + src1);
      *reinterpret_cast<uint4*>(Kout + static_cast<size_t>(slot) * a.row_bytes) = k0;
      *reinterpret_cast<uint4*>(Vout + static_cast<size_t>(slot) * a.row_bytes) = v0;
      *reinterpret_cast<uint4*>(Kout + static_cast<size_t>(other) * a.row_bytes) = k1;
      *reinterpret_cast<uint4*>(Vout + static_cast<size_t>(other) * a.row_bytes) = v1;
    }
  }
}

template <int ROW_BYTES>
__global__ __launch_bounds__(kGatherThreads) void prefill_gather(PrefillArgs a) {
  constexpr int LPR = ROW_BYTES / 16;
  constexpr int RPP = kGatherThreads / LPR;  // rows per pass
  const int u = blockIdx.y, tid = threadIdx.x;
  const int B = a.B;
  const int n = a.len[u];
  const int kept = n < B ? n : B;
  const int32_t* pos = a.pos + static_cast<size_t>(u) * B;
  const char* Kin = static_cast<const char*>(a.K) + static_cast<size_t>(u) * a.L_max * ROW_BYTES;
  const char* Vin = static_cast<const char*>(a.V) + static_cast<size_t>(u) * a.L_max * ROW_BYTES;
  char* Kout = static_cast<char*>(a.K_cache) + static_cast<size_t>(u) * B * ROW_BYTES;
  char* Vout = static_cast<char*>(a.V_cache) + static_cast<size_t>(u) * B * ROW_BYTES;
  const int r = tid / LPR, c = tid % LPR;
  const int first = blockIdx.x * kGatherRows;
  const int last = min(kept, first + kGatherRows);
  for (int slot = first + r; slot < last; slot += RPP) {
    const int p = pos[slot];
    if (p < 0 || p >= n) continue;  // never read outside the prompt, whatever pos[] holds
    const size_t src = static_cast<size_t>(p) * ROW_BYTES + c * 16;
    const size_t dst = static_cast<size_t>(slot) * ROW_BYTES + c * 16;
    *reinterpret_cast<uint4*>(Kout + dst) = load16_streaming(Kin + src);  // prompt rows are not needed again
    *reinterpret_cast<uint4*>(Vout + dst) = load16_streaming(Vin + src);
  }
}

// Which cached tokens survive one eviction step that shrinks a unit to `keep` tokens: the closed form of the
// rule above on the statistics as they stand, nothing modified.  mask[u][j] = 1 for survivors, 0 for victims and
// for empty slots.
__global__ __launch_bounds__(kSelThreads) void select_retained(DecodeArgs a, int keep, int32_t* mask_out) {
  constexpr int NT = kSelThreads;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds_keys[];  // [2][B] when B <= kMaxDecodeBudgetLds
  __shared__ __attribute__((aligned(16))) uint32_t sel_sh[SelectLds<1>::kWords];
  const int u = blockIdx.x, tid = threadIdx.x;
  const int B = a.B;
  const int n = min(a.n_used[u], B);
  const float* acc = a.stats + static_cast<size_t>(u) * 3 * B;
  const float* acc2 = acc + B;
  const float* cnt = acc2 + B;
  const int32_t* pos = a.pos + static_cast<size_t>(u) * B;
  int32_t* mask = mask_out + static_cast<size_t>(u) * B;
  uint32_t* var_key = (B <= kMaxDecodeBudgetLds) ? lds_keys : a.keys + static_cast<size_t>(u) * 2 * B;
  uint32_t* mas_key = var_key + B;
  if (n <= keep) {
    for (int i = tid; i < B; i += NT) mask[i] = i < n ? 1 : 0;
    return;
  }
  const uint32_t E = static_cast<uint32_t>(n - keep);
  const uint32_t m = min(static_cast<uint32_t>(n), static_cast<uint32_t>(a.pol.scope_size(a.scope, n)) + E - 1u);
  const bool by_pos = a.pol.needs_pos();
  for (int i = tid; i < n; i += NT)
    ranking_keys(acc[i], acc2[i], cnt[i], by_pos ? pos[i] : 0, a.pol, mas_key[i], var_key[i]);
  __syncthreads();
  const KSmallest scope = select_k_smallest<NT, 1, 1>([&](int i) { return var_key[i]; }, n, m, a.pol.scope_is_window(), sel_sh);
  auto key2 = [&](int i) -> uint32_t { return scope.has(var_key[i], i) ? mas_key[i] : 0xffffffffu; };
  const KSmallest out = select_k_smallest<NT, 1, 1>(key2, n, E, false, sel_sh);
  for (int i = tid; i < B; i += NT) mask[i] = (i < n && !out.has(key2(i), i)) ? 1 : 0;
}

// Overlap of two sets of cached tokens per unit (what section 4.1's consistency study compares): set X holds the
// positions pos_x[j] of the slots j < n_x with mask_x[j] != 0 (no mask: every such slot).  Positions inside a cache
// are distinct, so |A and B| is the number of B's members whose bit A has set in an LDS bitmap over [0, max_pos).
__global__ __launch_bounds__(256) void set_overlap(int slots_a, const int32_t* pos_a, const int32_t* mask_a,
                                                   const int32_t* n_a, int slots_b, const int32_t* pos_b,
                                                   const int32_t* mask_b, const int32_t* n_b, int max_pos,
                                                   int32_t* inter_out, int32_t* union_out) {
  extern __shared__ uint32_t bits[];  // (max_pos + 31) / 32 words, then the three counters
  const int u = blockIdx.x, tid = threadIdx.x;
  const int words = (max_pos + 31) / 32;
  uint32_t* const cnt = bits + words;  // |A|, |B|, |A and B|
  for (int i = tid; i < words; i += 256) bits[i] = 0u;
  if (tid < 3) cnt[tid] = 0u;
  __syncthreads();
  const int na = min(n_a[u], slots_a), nb = min(n_b[u], slots_b);
  uint32_t mine_a = 0, mine_b = 0, mine_i = 0;
  for (int j = tid; j < na; j += 256) {
    const int p = pos_a[static_cast<size_t>(u) * slots_a + j];
    if ((mask_a == nullptr || mask_a[static_cast<size_t>(u) * slots_a + j] != 0) && p >= 0 && p < max_pos) {
      atomicOr(&bits[p >> 5], 1u << (p & 31));
      ++mine_a;
    }
  }
  __syncthreads();
  for (int j = tid; j < nb; j += 256) {
    const int p = pos_b[static_cast<size_t>(u) * slots_b + j];
    if ((mask_b == nullptr || mask_b[static_cast<size_t>(u) * slots_b + j] != 0) && p >= 0 && p < max_pos) {
      ++mine_b;
      mine_i += (bits[p >> 5] >> (p & 31)) & 1u;
    }
  }
  atomicAdd(&cnt[0], mine_a);
  atomicAdd(&cnt[1], mine_b);
  atomicAdd(&cnt[2], mine_i);
  __syncthreads();
  if (tid == 0) {
    inter_out[u] = static_cast<int32_t>(cnt[2]);
    union_out[u] = static_cast<int32_t>(cnt[0] + cnt[1] - cnt[2]);
  }
}

}  // namespace

hipError_t launch_set_overlap(int units, int slots_a, const int32_t* pos_a, const int32_t* mask_a, const int32_t* n_a,
                              int slots_b, const int32_t* pos_b, const int32_t* mask_b, const int32_t* n_b, int max_pos,
                              int32_t* inter, int32_t* uni, hipStream_t s) {
  // the bitmap (the host keeps it within 64 KiB) and three counters: the largest range needs the raised limit
  const size_t lds = (static_cast<size_t>((max_pos + 31) / 32) + 3) * sizeof(uint32_t);
  if (!allow_key_lds(reinterpret_cast<const void*>(set_overlap), lds)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(set_overlap, dim3(units), dim3(256), lds, s, slots_a, pos_a, mask_a, n_a, slots_b, pos_b, mask_b, n_b,
                     max_pos, inter, uni);
  return hipGetLastError();
}

hipError_t launch_select_retained(const DecodeArgs& a, int keep, int32_t* mask, hipStream_t s) {
  const size_t lds = key_lds_bytes(a.B);
  if (!allow_key_lds(reinterpret_cast<const void*>(select_retained), lds)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(select_retained, dim3(a.units), dim3(kSelThreads), lds, s, a, keep, mask);
  return hipGetLastError();
}

// Copying the rows in the selection saves a launch (2 us of host time, 4 us of the GPU's) and costs what one compute unit takes
// for a unit's rows.  Whole call, us, in the selection against a kernel of its own, by KiB of K and V kept per unit: 32 (1 unit)
// 15.8 / 19.0, 64 (165 units) 45.5 / 56.4, 138 (3) 23.3 / 25.6, 159 (34) 40.5 / 44.7, 250 (96) 102.9 / 109, but 364 (1) 103.7 /
// 98.0 and 479 (3) 54.8 / 50.3.
static bool gathers_in_selection(const PrefillArgs& a) { return 2ll * a.B * a.row_bytes <= 256 << 10; }

// Whether a selection takes 512 threads instead of 1024.  Its searches are then of one digit behind four barriers (see fine_select), and a
// barrier is one of 8 waves; but a compute unit that has one workgroup then has half of the loads in flight.  Whole calls in us, 1024 / 512:
// up to 512 tokens 4 units x 256 of fp32 / 64 with output 24.6 / 23.1, 1 x 100 17.9 / 17.2, 300 x 300 of bf16 / 64 39.0 / 35.8, 2000 x 300
// 166 / 150; longer ones 24 x 966 32.4 / 33.1, 32 x 2048 82.4 / 83.7 (256 threads: 91.0), but where units outnumber the compute units
// 538 x 738 137.6 / 131.1, 1100 x 1024 364.7 / 356.7, 520 x 2000 550.5 / 545.4; 512 x 3072 1411 / 1416.
// ROCO_SELECT_THREADS=512, 1024: that many (the tests run both).
static bool few_threads_select(const PrefillArgs& a) {
  const char* const asked = getenv("ROCO_SELECT_THREADS");
  if (asked != nullptr && *asked != 0) return asked[0] == '5';
  return a.L_max <= 512 || (a.units > 256 && a.L_max <= 2048);
}

hipError_t launch_prefill_select_compact(int dtype, int head_dim, PrefillArgs a, hipStream_t s) {
  const int row_bytes = head_dim * (dtype == kBF16 ? 2 : 4);
  a.row_bytes = row_bytes;
  const bool gathered = key_lds_bytes(a.L_max) != 0 && gathers_in_selection(a);
  {
    ProfScope ps(kProfPrefillSelect, s);
    const size_t key_lds = key_lds_bytes(a.L_max);
    if (key_lds != 0) {
      const auto launch = [&](auto threads) {
        constexpr int NT = decltype(threads)::value;
        const auto kernel = gathered ? (a.shares_to_add > 2 ? prefill_select<2, true, true, NT> : prefill_select<2, false, true, NT>)
                                     : (a.shares_to_add > 2 ? prefill_select<2, true, false, NT> : prefill_select<2, false, false, NT>);
        if (!allow_key_lds(reinterpret_cast<const void*>(kernel), key_lds)) return false;
        hipLaunchKernelGGL(kernel, dim3(a.units), dim3(NT), key_lds, s, a);
        return true;
      };
      const bool launched = few_threads_select(a) ? launch(std::integral_constant<int, 512>{}) : launch(std::integral_constant<int, kSelThreads>{});
      if (!launched) return hipErrorInvalidValue;
    } else if (a.L_max <= 2 * kMaxDecodeBudgetLds) {  // one key per token still fits (40 units x 32768 tokens: 125 us against 200)
      const size_t one = static_cast<size_t>(a.L_max) * sizeof(uint32_t);
      if (!allow_key_lds(reinterpret_cast<const void*>(prefill_select<1, false, false>), one)) return hipErrorInvalidValue;
      hipLaunchKernelGGL((prefill_select<1, false, false>), dim3(a.units), dim3(kSelThreads), one, s, a);
    } else {
      hipLaunchKernelGGL((prefill_select<0, false, false>), dim3(a.units), dim3(kSelThreads), 0, s, a);
    }
  }
  if (gathered) return hipGetLastError();
  ProfScope ps(kProfPrefillGather, s);
  const dim3 grid((a.B + kGatherRows - 1) / kGatherRows, a.units);
  switch (row_bytes) {
    case 128: hipLaunchKernelGGL((prefill_gather<128>), grid, dim3(kGatherThreads), 0, s, a); break;
    case 256: hipLaunchKernelGGL((prefill_gather<256>), grid, dim3(kGatherThreads), 0, s, a); break;
    case 512: hipLaunchKernelGGL((prefill_gather<512>), grid, dim3(kGatherThreads), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace roco
