// Device helpers shared by the RoCo kernels (gfx950, 64-wide wavefronts).
#pragma once
#include "kernels.hpp"
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace roco {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;

enum : int { kF32 = 0, kBF16 = 1 };

// ---------------------------------------------------------------- element types
template <int DT> struct Elem;
template <> struct Elem<kF32> {
  using type = float;
  static constexpr int per16 = 4;  // elements in one 16-byte lane load
};
template <> struct Elem<kBF16> {
  using type = uint16_t;
  static constexpr int per16 = 8;
};

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}
// round to nearest even; inputs are finite attention outputs
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

template <int DT> __device__ __forceinline__ void unpack16(const uint4& w, float* f);
template <> __device__ __forceinline__ void unpack16<kF32>(const uint4& w, float* f) {
  f[0] = __uint_as_float(w.x); f[1] = __uint_as_float(w.y);
  f[2] = __uint_as_float(w.z); f[3] = __uint_as_float(w.w);
}
template <> __device__ __forceinline__ void unpack16<kBF16>(const uint4& w, float* f) {
  f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
  f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
  f[4] = __uint_as_float(w.z << 16); f[5] = __uint_as_float(w.z & 0xffff0000u);
  f[6] = __uint_as_float(w.w << 16); f[7] = __uint_as_float(w.w & 0xffff0000u);
}

template <int DT> __device__ __forceinline__ void store_elem(void* base, size_t idx, float v);
template <> __device__ __forceinline__ void store_elem<kF32>(void* base, size_t idx, float v) {
  static_cast<float*>(base)[idx] = v;
}
template <> __device__ __forceinline__ void store_elem<kBF16>(void* base, size_t idx, float v) {
  static_cast<uint16_t*>(base)[idx] = f32_to_bf16(v);
}

__device__ __forceinline__ uint4 load16(const void* p) { return *static_cast<const uint4*>(p); }
// Streaming variant: data that is touched once per kernel and should not displace what the caches hold.
typedef uint32_t uint4_vec __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load16_streaming(const void* p) {
  const uint4_vec v = __builtin_nontemporal_load(static_cast<const uint4_vec*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// The thread's index for code behind a kernel's main loop: what is derived from it is computed there, not kept in registers
// through the loop.
__device__ __forceinline__ int late_thread_id() {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  return tid;
}

// ---------------------------------------------------------------- cross-lane
// Lane exchange inside a 16-lane row through the data-parallel-primitive path of the vector ALU (no LDS
// traffic).  CTRL: 0xB1 = swap neighbours, 0x4E = swap pairs, 0x141 = mirror each 8 lanes, 0x140 = mirror
// each 16 lanes.  After the two swaps every lane of a quad holds the quad's value, so the two mirrors act
// as the xor-4 and xor-8 steps of a butterfly.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// All-reduce (sum) over aligned groups of LANES lanes (LANES a power of two <= 64).
template <int LANES> __device__ __forceinline__ float group_sum(float v) {
  if (LANES >= 2) v += dpp_move<0xB1>(v);
  if (LANES >= 4) v += dpp_move<0x4E>(v);
  if (LANES >= 8) v += dpp_move<0x141>(v);
  if (LANES >= 16) v += dpp_move<0x140>(v);
#pragma unroll
  for (int m = 16; m < LANES; m <<= 1) v += __shfl_xor(v, m, kWave);
  return v;
}
template <int LANES> __device__ __forceinline__ float group_max(float v) {
#pragma unroll
  for (int m = 1; m < LANES; m <<= 1) v = fmaxf(v, __shfl_xor(v, m, kWave));
  return v;
}

// Inclusive prefix sum over the 64 lanes of a wave on the vector ALU's lane-shift path: four shifted adds inside
// each row of 16 lanes, then the last lane of rows 0 and 2 is added to rows 1 and 3, then lane 31 to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  auto shr = [](uint32_t x, auto ctrl, auto row_mask) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(x), decltype(ctrl)::value, decltype(row_mask)::value, 0xF, false));
  };
  using std::integral_constant;
  v += shr(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});  // row_shr:1
  v += shr(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});  // row_shr:2
  v += shr(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});  // row_shr:4
  v += shr(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});  // row_shr:8
  v += shr(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});  // row_bcast:15 into rows 1, 3
  v += shr(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});  // row_bcast:31 into rows 2, 3
  return v;
}

// Minimum over the 64 lanes of a wave, the same way.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  auto other = [](uint32_t x, auto ctrl, auto row_mask) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(-1, static_cast<int>(x), decltype(ctrl)::value, decltype(row_mask)::value, 0xF, false));
  };
  using std::integral_constant;
  v = min(v, other(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{}));
  v = min(v, other(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{}));
  v = min(v, other(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{}));
  v = min(v, other(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{}));
  v = min(v, other(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{}));
  v = min(v, other(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{}));
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), kWave - 1));
}

// Bitwise or over the 64 lanes of a wave, the same way.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  auto other = [](uint32_t x, auto ctrl, auto row_mask) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(x), decltype(ctrl)::value, decltype(row_mask)::value, 0xF, false));
  };
  using std::integral_constant;
  v |= other(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});
  v |= other(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
  v |= other(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
  v |= other(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
  v |= other(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});
  v |= other(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), kWave - 1));
}

// Index of the smallest key over all threads of the block (the lowest index among equal keys): every thread brings its
// own best and gets the answer.  `sh` needs one entry per wave.  The waves' minima are reduced by the code that made them.
template <int NT> __device__ __forceinline__ uint32_t block_argmin(uint32_t key, uint32_t idx, uint2* sh) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll 1
  for (int round = 0;; ++round) {
    const uint32_t k = wave_min(key);
    const uint32_t i = wave_min(key == k ? idx : 0xffffffffu);
    if (round == 1) return i;
    if (lane == 0) sh[threadIdx.x / kWave] = make_uint2(k, i);
    __syncthreads();
    const uint2 v = lane < NT / kWave ? sh[lane] : make_uint2(0xffffffffu, 0xffffffffu);
    key = v.x;
    idx = v.y;
  }
}

// Exclusive prefix sum of one value per thread over the whole block, in thread order.
// `sh` needs NT/64 + 1 words; returns the block total through `total`.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* sh, uint32_t& total) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  uint32_t incl = wave_inclusive_scan(v);
  __syncthreads();  // protects `sh` against readers of a previous call
  if (lane == kWave - 1) sh[wave] = incl;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) {
    uint32_t s = sh[w];
    if (w < wave) off += s;
    tot += s;
  }
  total = tot;
  return off + incl - v;
}

// ---------------------------------------------------------------- k-smallest selection
// Non-negative IEEE floats order like their bit patterns read as uint32, so selection runs on
// integers and is exact.  radix_select finds the k-th smallest key (k is 1-based, 1 <= k <= n) among
// key_of(0..n-1), digits of up to 11 bits from the top; it also returns how many keys are strictly smaller and how
// many are equal.  What it costs is its barriers and its passes over the keys, so the first digit is wide: the exponent and
// the three leading mantissa bits (no key has the top bit, but the mark and, under `small`, negative positions) spread a
// unit's variances or scores over bins of an eighth of an octave, and usually few enough keys share the chosen one that no
// second digit is counted -- as soon as a bin holds at most kSelectRanked keys they are gathered and searched without another
// barrier.  A thread clears the bins it owns while it reads them, so a digit takes three barriers.
// AHEAD: keys per thread that a pass requests before it uses the first: four where they come from memory, and from LDS with few
// threads (the step of 512 units x 2048 slots of bf16 / 128: 95.6 -> 94.1 us); with 1024 threads other waves fill the time, and
// the longer code has to be fetched.
// The largest key, 0xffffffff, is the mark of elements that do not take part: it is neither counted (thousands of additions
// to one bin would be served one after the other) nor gathered.
// `small`: the keys are small numbers, positions or indices: the digits then start at the highest bit that is set in any of
// them, which takes one more pass over the keys.  From the top they would all share the first bins, whose counts are served
// one key after the other, and the search among the last candidates would walk through twenty empty bits (step of 4 heads on
// 300 units x 64 slots under a window scope: 23.7 -> 16.9 us; 16 tokens on 64 units x 512 slots: 41.8 -> 33.8).
// PER_WORD: bins in a word of LDS, 2 for up to 65535 keys.  It costs half a percent of a small step, but where the units'
// ranking keys fill the LDS four KiB of it are a resident workgroup (decode step of bf16 / 128 with 512 units x 9400 slots 484
// -> 459 us, 768 x 6000 453 -> 438).
// `sh` needs SelectLds<PER_WORD>::kWords words of LDS.  All threads of the block call it.
constexpr int kSelectBins = 2048;
constexpr int kSelectRanked = 128;
template <int PER_WORD> struct SelectLds {
  static constexpr int kBinWords = kSelectBins / PER_WORD;
  static constexpr int kWords = kBinWords + 16 + 8;
};
static_assert(kSelectRanked == 2 * kWave, "two candidates per lane");

// f(key) for every key of this thread, in no particular order.
template <int NT, int AHEAD, class KeyFn, class F>
__device__ __forceinline__ void for_each_key(KeyFn key_of, int n, int tid, F f) {
  if (AHEAD == 1 || n <= NT) {
#pragma unroll 1
    for (int i = tid; i < n; i += NT) f(key_of(i));
    return;
  }
#pragma unroll 1
  for (int i = tid; i < n; i += AHEAD * NT) {
    uint32_t key[AHEAD];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) key[j] = key_of(min(i + j * NT, n - 1));
#pragma unroll
    for (int j = 0; j < AHEAD; ++j)
      if (i + j * NT < n) f(key[j]);
  }
}

template <int NT, int PER_WORD, int AHEAD, class KeyFn>
__device__ __forceinline__ void radix_select(KeyFn key_of, int n, uint32_t k, bool small, uint32_t* sh,
                             uint32_t& kth, uint32_t& n_less, uint32_t& n_equal) {
  static_assert(NT <= 1024 && kSelectBins % NT == 0, "whole bins per thread");
  constexpr int OWN = kSelectBins / NT;   // consecutive bins per thread
  static_assert(PER_WORD == 1 || (PER_WORD == 2 && OWN % 2 == 0), "whole words per thread");
  constexpr int OWN_WORDS = OWN / PER_WORD;
  uint32_t* const wtot = sh + SelectLds<PER_WORD>::kBinWords;  // totals of the waves' bins
  uint32_t* const res = wtot + 16;                // bin, keys below the bin, keys in the bin, candidates gathered
  const int tid = late_thread_id(), lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  __syncthreads();  // `sh` may still be in use by a previous call
#pragma unroll
  for (int i = 0; i < OWN_WORDS; ++i) sh[tid * OWN_WORDS + i] = 0;
  if (small) {
    uint32_t any = 0;
    for_each_key<NT, AHEAD>(key_of, n, tid, [&](uint32_t key) { any |= key != 0xffffffffu ? key : 0u; });
    any = wave_or(any);
    if (lane == 0) wtot[wave] = any;
  }
  __syncthreads();
  int top = 31;  // bits that are still to be counted
  if (small) top = 32 - __builtin_clz(wave_or(lane < NT / kWave ? wtot[lane] : 0u) | 1u);
  uint32_t prefix = 0, mask = 0, kk = k, less = 0, neq = 0;
  auto takes_part = [&](uint32_t key) { return (key & mask) == prefix && key != 0xffffffffu; };
#pragma unroll 1
  while (top > 0) {
    const int shift = max(top - 11, 0);
    const uint32_t digit = (1u << (top - shift)) - 1u;
    top = shift;
    for_each_key<NT, AHEAD>(key_of, n, tid, [&](uint32_t key) {
      const uint32_t bin = (key >> shift) & digit;
      if (takes_part(key)) atomicAdd(&sh[bin / PER_WORD], PER_WORD == 2 ? 1u << (16 * (bin & 1)) : 1u);
    });
    __syncthreads();
    uint32_t h[OWN], sum = 0;
#pragma unroll
    for (int i = 0; i < OWN_WORDS; ++i) {
      const uint32_t word = sh[tid * OWN_WORDS + i];
      sh[tid * OWN_WORDS + i] = 0;  // ready for the next digit
      h[PER_WORD * i] = PER_WORD == 2 ? word & 0xffffu : word;
      if (PER_WORD == 2) h[PER_WORD * i + PER_WORD - 1] = word >> 16;
    }
#pragma unroll
    for (int i = 0; i < OWN; ++i) sum += h[i];
    uint32_t excl = wave_inclusive_scan(sum);
    if (lane == kWave - 1) wtot[wave] = excl;
    excl -= sum;
    __syncthreads();
    {  // the totals of the waves before this one: one read, one scan
      const uint32_t t = wave_inclusive_scan(lane < NT / kWave ? wtot[lane] : 0u);
      if (wave > 0) excl += __builtin_amdgcn_readlane(t, wave - 1);
      const uint32_t counted = __builtin_amdgcn_readlane(t, NT / kWave - 1);
      if (kk > counted) {  // among the keys that are not counted (first digit only: later ones lie inside a counted bin)
        kth = 0xffffffffu;
        n_less = counted;
        n_equal = n - counted;
        return;
      }
    }
    if (excl < kk && kk <= excl + sum) {  // the chosen bin is one of this thread's
#pragma unroll
      for (int i = 0; i < OWN; ++i) {
        if (excl < kk && kk <= excl + h[i]) { res[0] = tid * OWN + i; res[1] = excl; res[2] = h[i]; res[3] = 0; }
        excl += h[i];
      }
    }
    __syncthreads();
    prefix |= res[0] << shift;
    mask |= digit << shift;
    less += res[1];
    kk -= res[1];
    neq = res[2];
    if (neq <= kSelectRanked && shift > 0) {
      // Few candidates are left: they are gathered (into the bins, which are clear and not needed any more), and a wave
      // finishes on its own, two candidates per lane, bit by bit from the top of what is left of the keys: the candidates
      // with a zero there are the lower ones.  Ballots and scalar counts only, and the search ends as soon as one candidate
      // is left.  Up to four waves all do this, without a barrier; more would share the schedulers with one another, so
      // the first one leaves the answer to the others (16 tokens on 64 units x 512 slots: 35.3 -> 32.4 us).
      constexpr bool kOneWave = NT > 4 * kWave;
      for_each_key<NT, AHEAD>(key_of, n, tid, [&](uint32_t key) {
        if (takes_part(key)) sh[atomicAdd(&res[3], 1u)] = key;
      });
      __syncthreads();
      if (!kOneWave || wave == 0) {
        const uint32_t c0 = sh[lane], c1 = sh[lane + kWave];
        uint64_t in0 = neq >= 64 ? ~0ull : (1ull << neq) - 1ull;
        uint64_t in1 = neq > 64 ? (neq == 128 ? ~0ull : (1ull << (neq - 64)) - 1ull) : 0ull;
        uint32_t left = neq;
#pragma unroll 1
        for (int bit = shift - 1; bit >= 0 && left > 1; --bit) {
          const uint64_t z0 = in0 & ~__builtin_amdgcn_ballot_w64((c0 >> bit) & 1u);
          const uint64_t z1 = in1 & ~__builtin_amdgcn_ballot_w64((c1 >> bit) & 1u);
          const uint32_t zeros = __builtin_popcountll(z0) + __builtin_popcountll(z1);
          if (kk <= zeros) {
            in0 = z0; in1 = z1; left = zeros;
          } else {
            in0 &= ~z0; in1 &= ~z1; left -= zeros;
            kk -= zeros; less += zeros;
          }
        }
        prefix = in0 != 0 ? __builtin_amdgcn_readlane(c0, __builtin_ctzll(in0))
                          : __builtin_amdgcn_readlane(c1, __builtin_ctzll(in1));
        neq = left;
        if (kOneWave && lane == 0) { res[0] = prefix; res[1] = less; res[2] = neq; }
      }
      if (kOneWave) {
        __syncthreads();
        prefix = res[0];
        less = res[1];
        neq = res[2];
      }
      break;
    }
  }
  kth = prefix;
  n_less = less;
  n_equal = neq;
}

// The k smallest keys, equal keys taken in index order: element i is selected iff
//   key < kth  ||  (key == kth && i <= index_limit).
struct KSmallest {
  uint32_t kth;
  uint32_t index_limit;
  __device__ __forceinline__ bool has(uint32_t key, uint32_t i) const {
    return key < kth || (key == kth && i <= index_limit);
  }
};

// Up to kCountedKeys keys are not searched: the threads count for every key how many do not follow it, and the one that counts k
// is the last of the k smallest.  Two instructions per pair of keys instead of four barriers, the bins and the chain of the search
// among the last candidates (128 keys in four waves: 4800 -> 3100 cycles).  256 keys in sixteen waves take as long either way,
// and on a compute unit that has several units' searches at a time longer (block_prepare of 674 units x 196 slots 10.8 -> 13.7 us).
// Keys that are equal come in the order of their blocks of 64; inside a block they all count the same number, so if the boundary
// falls among such keys nobody counts k: false, and the search has to say which of them belong.
constexpr int kCountedKeys = 2 * kWave;
template <int NT, class KeyFn>
__device__ __forceinline__ bool count_k_smallest(KeyFn key_of, int n, uint32_t k, uint32_t* sh, KSmallest& r) {
  constexpr int PARTS = NT / kCountedKeys;      // threads that share the counting for a key
  constexpr int SHARE = kCountedKeys / PARTS;   // keys of each
  static_assert(PARTS > 1 && kWave % SHARE == 0 && SHARE % 4 == 0, "a share lies in one block of keys");
  uint32_t* const counts = sh + kCountedKeys;
  uint32_t* const res = counts + kCountedKeys;  // the key, 1 + its index
  const int tid = late_thread_id(), mine = tid & (kCountedKeys - 1);
  const int first = __builtin_amdgcn_readfirstlane(tid / kCountedKeys) * SHARE;
  const bool earlier = first / kWave <= __builtin_amdgcn_readfirstlane(mine / kWave);  // (or the key's own block)
  __syncthreads();  // `sh` may still be in use by a previous call
  if (tid < kCountedKeys) {
    sh[tid] = tid < n ? key_of(tid) : 0xffffffffu;
    counts[tid] = 0;
  }
  if (tid == 0) res[1] = 0;
  __syncthreads();
  const uint32_t key = sh[mine];
  const uint4* const others = reinterpret_cast<const uint4*>(sh + first);
  uint32_t count = 0;
  if (earlier) {
#pragma unroll 4
    for (int j = 0; j < SHARE / 4; ++j) {
      const uint4 o = others[j];
      count += (o.x <= key) + (o.y <= key) + (o.z <= key) + (o.w <= key);
    }
  } else {
#pragma unroll 4
    for (int j = 0; j < SHARE / 4; ++j) {
      const uint4 o = others[j];
      count += (o.x < key) + (o.y < key) + (o.z < key) + (o.w < key);
    }
  }
  atomicAdd(&counts[mine], count);
  __syncthreads();
  if (tid < n && counts[mine] == k && key != 0xffffffffu) {  // (n is at most kCountedKeys)
    res[0] = key;
    atomicMax(&res[1], static_cast<uint32_t>(mine) + 1u);
  }
  __syncthreads();
  if (res[1] == 0) return false;
  r = KSmallest{res[0], res[1] - 1u};
  return true;
}

// Where the ranking keys usually lie, between 2^-52 and 2^12, one digit of 1/32 of an octave leaves so few candidates that no second one
// has to be counted (1/16, with half of the bins, does not: such searches end here in vain), and its 2048 bins, two to a word, are few
// enough for up to eight waves to scan them each by itself: four barriers instead of eight.  Cycles for the 65th / 1024th of 2048 keys:
// 256 threads 7670 / 7220 -> 6390 / 5840, 512 threads 6900 / 6400 -> 6160 / 5200; 1024 threads 6430 / 5480 -> 5960 / 5150, which the
// sixteen waves' scans make up for with fewer keys, and decode_finish lost half a microsecond by the longer code.  What is left are
// the additions to the bins, served a few at a time.  Steps: 128 units x 4 heads x 2048 slots 38.4 -> 37.7 us, 512 x 16 tokens x
// 2048 110.6 -> 109.1.
// False if the k-th smallest key lies outside or among more than kSelectRanked candidates: then the search above has to find it.
constexpr int kFineBins = 2048, kFineShift = 18;
constexpr uint32_t kFineFrom = (127u - 52u) << 23;
template <int NT, int PER_WORD, int AHEAD, class KeyFn>
__device__ __forceinline__ bool fine_select(KeyFn key_of, int n, uint32_t k, uint32_t* sh, uint32_t& kth, uint32_t& n_less, uint32_t& n_equal) {
  // The candidates have words of their own where bins of a word each leave them; else they take bins that have been read, behind one
  // barrier more: with words of their own the one-kernel decode step would lose its third workgroup at the largest budgets.
  constexpr bool kOwnWords = kFineBins / 2 + 4 + kSelectRanked <= SelectLds<PER_WORD>::kWords;
  uint32_t* const res = sh + kFineBins / 2;  // candidates gathered; the key, keys below it, keys equal to it
  uint32_t* const list = kOwnWords ? res + 4 : sh;
  static_assert(kFineBins / 2 + 4 <= SelectLds<PER_WORD>::kWords && kSelectRanked <= kFineBins / 2, "the bins and four words");
  const int tid = late_thread_id(), lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  auto bin_of = [](uint32_t key) { return min((max(key, kFineFrom) - kFineFrom) >> kFineShift, static_cast<uint32_t>(kFineBins - 1)); };
  __syncthreads();  // `sh` may still be in use by a previous call
  if (tid < kFineBins / 8) *reinterpret_cast<uint4*>(sh + 4 * tid) = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) res[0] = 0;
  __syncthreads();
  for_each_key<NT, AHEAD>(key_of, n, tid, [&](uint32_t key) {
    const uint32_t bin = bin_of(key);
    if (key != 0xffffffffu) atomicAdd(&sh[bin >> 1], 1u << (16 * (bin & 1)));
  });
  __syncthreads();
  // 32 bins per lane
  uint32_t pairs = 0;  // (at most 65535 keys)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint4 w = *reinterpret_cast<const uint4*>(sh + 16 * lane + 4 * i);
    pairs += w.x + w.y + w.z + w.w;
  }
  const uint32_t mine = (pairs & 0xffffu) + (pairs >> 16);
  const uint32_t upto = wave_inclusive_scan(mine);
  const uint64_t reach = __builtin_amdgcn_ballot_w64(upto >= k);
  if (reach == 0) return false;  // among the keys that are not counted
  const int owner = __builtin_ctzll(reach);
  uint32_t less = __builtin_amdgcn_readlane(upto - mine, owner);
  const uint32_t word = sh[16 * owner + ((lane & 31) >> 1)];
  const uint32_t count = lane < 32 ? ((lane & 1) ? word >> 16 : word & 0xffffu) : 0u;
  const uint32_t inside = wave_inclusive_scan(count);
  const int off = __builtin_ctzll(__builtin_amdgcn_ballot_w64(less + inside >= k));
  const uint32_t cand = __builtin_amdgcn_readlane(count, off);
  less += __builtin_amdgcn_readlane(inside, off) - cand;
  const uint32_t bin = static_cast<uint32_t>(32 * owner + off);
  if (bin == 0 || bin == kFineBins - 1 || cand > kSelectRanked) return false;
  if (!kOwnWords) __syncthreads();  // every wave has read the bins
  for_each_key<NT, AHEAD>(key_of, n, tid, [&](uint32_t key) {
    if (bin_of(key) == bin && key != 0xffffffffu) list[atomicAdd(&res[0], 1u)] = key;
  });
  __syncthreads();
  constexpr bool kOneWave = NT > 4 * kWave;  // (as above)
  uint32_t kk = k - less, left = cand;
  if (!kOneWave || wave == 0) {
    const uint32_t c0 = list[lane], c1 = list[lane + kWave];
    uint64_t in0 = cand >= 64 ? ~0ull : (1ull << cand) - 1ull;
    uint64_t in1 = cand > 64 ? (cand == 128 ? ~0ull : (1ull << (cand - 64)) - 1ull) : 0ull;
#pragma unroll 1
    for (int bit = kFineShift - 1; bit >= 0 && left > 1; --bit) {
      const uint64_t z0 = in0 & ~__builtin_amdgcn_ballot_w64((c0 >> bit) & 1u);
      const uint64_t z1 = in1 & ~__builtin_amdgcn_ballot_w64((c1 >> bit) & 1u);
      const uint32_t zeros = __builtin_popcountll(z0) + __builtin_popcountll(z1);
      if (kk <= zeros) {
        in0 = z0; in1 = z1; left = zeros;
      } else {
        in0 &= ~z0; in1 &= ~z1; left -= zeros;
        kk -= zeros; less += zeros;
      }
    }
    kth = in0 != 0 ? __builtin_amdgcn_readlane(c0, __builtin_ctzll(in0)) : __builtin_amdgcn_readlane(c1, __builtin_ctzll(in1));
    if (kOneWave && lane == 0) { res[1] = kth; res[2] = less; res[3] = left; }
  }
  if (kOneWave) {
    __syncthreads();
    kth = res[1];
    less = res[2];
    left = res[3];
  }
  n_less = less;
  n_equal = left;
  return true;
}

// FINE, spread: the keys may lie where fine_select finds them.  Positions and counts do not (a prompt of 1207 tokens under an oldest-first
// policy lost 0.5 us to searches in vain), and a search that is hardly ever made is not worth the code.
template <int NT, int PER_WORD, int AHEAD, bool FINE = true, class KeyFn>
__device__ __forceinline__ KSmallest select_k_smallest(KeyFn key_of, int n, uint32_t k, bool small, uint32_t* sh, bool spread = true) {
  // everything is wanted (the policies whose scope is the whole cache, say): nothing to select
  if (k >= static_cast<uint32_t>(n)) return KSmallest{0xffffffffu, 0xffffffffu};
  // At most two rounds through one copy of the search (these kernels start cold: a second copy is instructions to fetch):
  // the k-th smallest key, then, if ties straddle the boundary, which of the equal keys belong: the lowest indices.
  KSmallest r = {0u, 0xffffffffu};
  if (n <= kCountedKeys && count_k_smallest<NT>(key_of, n, k, sh, r)) return r;
  uint32_t take = k;
#pragma unroll 1
  for (int round = 0; round < 2; ++round) {
    const uint32_t kth = r.kth;
    uint32_t found, n_less, n_equal;
    bool done = false;
    if constexpr (FINE && NT <= 512) done = round == 0 && spread && !small && n <= 65535 && fine_select<NT, PER_WORD, AHEAD>(key_of, n, take, sh, found, n_less, n_equal);
    if (!done)
      radix_select<NT, PER_WORD, AHEAD>(
          [&](int i) {
            const uint32_t key = key_of(i);
            return round == 0 ? key : key == kth ? static_cast<uint32_t>(i) : 0xffffffffu;
          },
          n, take, round == 1 || small, sh, found, n_less, n_equal);
    if (round == 1) {
      r.index_limit = found;
    } else {
      r.kth = found;
      take = k - n_less;  // how many of the keys equal to kth belong to the selection
      if (take == n_equal) break;
    }
  }
  return r;
}

// Scope = `scope` lowest variance keys among [0, B); returns the slot of lowest MAS key inside it (lowest
// slot on equal keys).  Every thread of the block calls it and gets the same answer.
template <int NT, int PER_WORD, bool FINE = true, class VarFn, class MasFn>
__device__ __forceinline__ int select_victim(VarFn var_key_of, MasFn mas_key_of, int B, const Policy& pol, int scope, uint32_t* sel_sh,
                                             uint2* best_sh) {
  const int tid = late_thread_id();
  const KSmallest sc = select_k_smallest<NT, PER_WORD, NT <= 4 * kWave ? 4 : 1, FINE>(var_key_of, B,
                                             static_cast<uint32_t>(pol.scope_size(scope, B)), pol.scope_is_window(), sel_sh);
  uint32_t key = 0xffffffffu, idx = 0xffffffffu;
#pragma unroll 1
  for (int i = tid; i < B; i += NT) {
    if (sc.has(var_key_of(i), i)) {
      const uint32_t k = mas_key_of(i);
      if (k < key || idx == 0xffffffffu) { key = k; idx = static_cast<uint32_t>(i); }
    }
  }
  return static_cast<int>(block_argmin<NT>(key, idx, best_sh));
}
template <int NT, int PER_WORD>
__device__ __forceinline__ int select_victim_block(const uint32_t* var_key, const uint32_t* mas_key, int B, const Policy& pol, int scope,
                                                   uint32_t* sel_sh, uint2* best_sh) {
  return select_victim<NT, PER_WORD>([&](int i) { return var_key[i]; }, [&](int i) { return mas_key[i]; }, B, pol, scope, sel_sh, best_sh);
}

// Ranking keys of one cached token: the token of lowest importance key among the tokens of lowest scope key
// is evicted; keys are compared as unsigned integers (non-negative floats order like their bit patterns).
// For RoCo these are the mean attention score and the attention variance, each operation rounded on its own
// (no fused multiply-add), so that a single observation gives a variance of exactly zero:
//   MAS = Acc/Count,  Var = max(0, Acc2/Count - MAS^2)          (section 4.3 of the paper)
// A protected sink position gets the largest importance key without the top bit, which the search leaves out (so does a negative
// position, which is below any number of sinks); 0xffffffff is the marker that the selections use for "outside the scope".
// N tokens at a time: the policy is asked for once, and the divisions, chains of ten dependent instructions, run side by side.
template <int N>
__device__ __forceinline__ void ranking_keys(const float* acc, const float* acc2, const float* count, const int* pos,
                                             const Policy& pol, uint32_t* mas_key, uint32_t* var_key) {
  const bool by_variance = pol.scope_kind == kScopeStd;
  float mas[N];
  if (by_variance || pol.importance == kImpMas) {
#pragma unroll
    for (int e = 0; e < N; ++e) {
      mas[e] = __fdiv_rn(acc[e], count[e]);
      mas_key[e] = __float_as_uint(mas[e]) & 0x7fffffffu;
    }
  }
  if (by_variance) {
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const float ex2 = __fdiv_rn(acc2[e], count[e]);
      const float var = __fsub_rn(ex2, __fmul_rn(mas[e], mas[e]));
      var_key[e] = var > 0.0f ? __float_as_uint(var) : 0u;
    }
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) var_key[e] = pol.scope_kind == kScopeWindow ? static_cast<uint32_t>(pos[e]) : 0u;
  }
  if (pol.importance != kImpMas) {
    const bool oldest = pol.importance == kImpOldest, accumulated = pol.importance == kImpAas;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const float score = accumulated ? acc[e] : acc2[e];
      mas_key[e] = oldest ? (pos[e] < pol.sinks ? 0x7fffffffu : static_cast<uint32_t>(pos[e]))
                          : score > 0.0f ? __float_as_uint(score) : 0u;
    }
  }
}
__device__ __forceinline__ void ranking_keys(float acc, float acc2, float count, int pos, const Policy& pol,
                                             uint32_t& mas_key, uint32_t& var_key) {
  ranking_keys<1>(&acc, &acc2, &count, &pos, pol, &mas_key, &var_key);
}

}  // namespace roco
