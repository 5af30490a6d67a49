// Prefill attention statistics on the plain vector ALUs, for every supported dtype / head_dim.
//
// The path of prompts too small for the matrix cores to pay (see prefill_rows_are_tiny), of bf16 / 128 prompts above 4M
// tokens, and the cross-check for the matrix-core paths.
// Two passes, because a column statistic needs the final normaliser of every row it sums over:
//   pass 1: one wave per query row i streams keys 0..i with an online softmax and stores the row's base-2
//           log-sum-exp (and the attention output, if asked)                     (section 2.1, eq. 1; causal)
//   pass 2: one wave per key column j streams queries j..len-1, recomputes the logit and accumulates
//           Acc[j] = sum_i P[i,j] and Acc2[j] = sum_i P[i,j]^2 in fp32            (section 4.3)
// Count[j] = len - j has a closed form and is not accumulated.  The L x L matrix is never stored.
#include <cstdlib>

#include "kernels.hpp"
#include "profile.hpp"
#include "stream.hpp"

namespace roco {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kUnroll = 4;

// WPR waves share a query row, each with every WPR-th block of keys: one, or all four of a workgroup.  What bounds a prompt of few rows
// is the chain of a wave's trips to the L2, a block of 16 (bf16 / 64: 32) keys each; with more rows than the chip holds waves of, the
// merge costs more than the shorter chain gains (see launch_rows_t).
template <int DT, int D, int WPR>
__global__ __launch_bounds__(kThreads) void prefill_rows_simple(PrefillArgs a) {
  using G = RowGeom<DT, D>;
  static_assert(WPR == 1 || WPR == kWaves, "a row is one wave's or the workgroup's");
  const int uq = blockIdx.y;       // (unit, query head)
  const int uk = uq / a.group;     // the unit: its keys, values and length
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int c = lane % G::LPR;
  const int part = WPR == 1 ? 0 : wave;
  const int i = WPR == 1 ? blockIdx.x * kWaves + wave : blockIdx.x;
  const int len = a.len[uk];
  if (i >= len) return;
  const size_t ubase = static_cast<size_t>(uq) * a.L_max;
  const size_t kbase = static_cast<size_t>(uk) * a.L_max;
  float qf[G::EPL];
  unpack16<DT>(load16(static_cast<const char*>(a.Q) + (ubase + i) * G::ROW_BYTES + c * 16), qf);
#pragma unroll
  for (int e = 0; e < G::EPL; ++e) qf[e] *= a.scale_log2;
  const char* Kb = static_cast<const char*>(a.K) + kbase * G::ROW_BYTES;
  const char* Vb = static_cast<const char*>(a.V) + kbase * G::ROW_BYTES;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  FlashState<G::EPL> st;
  st.reset();
  auto bias = [&](int row, int) -> float { return (i - row < w) ? rb : 0.0f; };  // row <= i here
  auto fix = [](int, uint4&, int) {};
  constexpr int PASS = kUnroll * G::R;
  const int passes = (i + WPR * PASS - part * PASS) / (WPR * PASS);  // blocks of this wave, of keys up to i
  if (w > 0)
    stream_attend<DT, D, kUnroll, true, false>(qf, Kb, Vb, 0, i + 1, i + 1, passes, 0, WPR * PASS, part * PASS, bias, nullptr, nullptr, -1, fix, fix, [] {}, st);
  else
    stream_attend<DT, D, kUnroll, false, false>(qf, Kb, Vb, 0, i + 1, i + 1, passes, 0, WPR * PASS, part * PASS, bias, nullptr, nullptr, -1, fix, fix, [] {}, st);
  merge_groups_in_wave<DT, D>(st);
  if constexpr (WPR > 1) {  // the first wave merges the others, in their order
    __shared__ float part_s[WPR][G::LPR][G::EPL + 2];
    if (wave > 0 && lane < G::LPR) {
      float* const p = part_s[wave][lane];
      p[G::EPL] = st.m;
      p[G::EPL + 1] = st.l;
#pragma unroll
      for (int e = 0; e < G::EPL; ++e) p[e] = st.acc[e];
    }
    __syncthreads();
    if (wave > 0 || lane >= G::LPR) return;
#pragma unroll
    for (int k = 1; k < WPR; ++k) {
      const float* const p = part_s[k][lane];
      const float m_o = p[G::EPL], m_new = fmaxf(st.m, m_o);
      const float f0 = (st.m > -INFINITY) ? fast_exp2(st.m - m_new) : 0.0f, f1 = (m_o > -INFINITY) ? fast_exp2(m_o - m_new) : 0.0f;
      st.l = st.l * f0 + p[G::EPL + 1] * f1;
#pragma unroll
      for (int e = 0; e < G::EPL; ++e) st.acc[e] = st.acc[e] * f0 + p[e] * f1;
      st.m = m_new;
    }
  }
  if (lane == 0) a.lse[ubase + i] = st.m + log2f(st.l);
  if (a.O != nullptr && lane < G::LPR) {
    const float inv = 1.0f / st.l;
#pragma unroll
    for (int e = 0; e < G::EPL; ++e)
      store_elem<DT>(a.O, (ubase + i) * D + lane * G::EPL + e, st.acc[e] * inv);
  }
}

template <int DT, int D>
__global__ __launch_bounds__(kThreads) void prefill_columns_simple(PrefillArgs a) {
  using G = RowGeom<DT, D>;
  constexpr int U = kUnroll;
  const int u = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / G::LPR, c = lane % G::LPR;
  const int j = blockIdx.x * kWaves + wave;
  const int len = a.len[u];
  if (j >= len) return;
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  float kf[G::EPL];
  unpack16<DT>(load16(static_cast<const char*>(a.K) + (ubase + j) * G::ROW_BYTES + c * 16), kf);
#pragma unroll
  for (int e = 0; e < G::EPL; ++e) kf[e] *= a.scale_log2;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const float inv_heads = 1.0f / static_cast<float>(a.group);
  float s1 = 0.0f, s2 = 0.0f;
  for (int base = j; base < len; base += U * G::R) {
    float pbar[U];  // sum over the unit's query heads of P[row, j] (one head without grouped-query attention)
#pragma unroll
    for (int x = 0; x < U; ++x) pbar[x] = 0.0f;
    for (int h = 0; h < a.group; ++h) {
      const size_t qbase = (static_cast<size_t>(u) * a.group + h) * a.L_max;
      const char* Qb = static_cast<const char*>(a.Q) + qbase * G::ROW_BYTES;
      const float* lse = a.lse + qbase;
      uint4 qw[U];
      float ls[U];
#pragma unroll
      for (int x = 0; x < U; ++x) {
        const int row = base + x * G::R + g;
        const int r = row < len ? row : j;
        qw[x] = load16(Qb + static_cast<size_t>(r) * G::ROW_BYTES + c * 16);
        ls[x] = lse[r];
      }
#pragma unroll
      for (int x = 0; x < U; ++x) {
        const int row = base + x * G::R + g;
        float qf[G::EPL];
        unpack16<DT>(qw[x], qf);
        float dot = 0.0f;
#pragma unroll
        for (int e = 0; e < G::EPL; ++e) dot = fmaf(qf[e], kf[e], dot);
        dot = group_sum<G::LPR>(dot);
        if (row < len) {
          const float t = dot + ((row - j < w) ? rb : 0.0f);
          pbar[x] += exp2f(t - ls[x]);
        }
      }
    }
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const float p = pbar[x] * inv_heads;  // rows past the end contribute exactly zero
      s1 += p;
      if (a.pol.counts_above_average()) s2 += (p * static_cast<float>(base + x * G::R + g + 1) > 1.0f) ? 1.0f : 0.0f;
      else s2 = fmaf(p, p, s2);
    }
  }
#pragma unroll
  for (int m = G::LPR; m < kWave; m <<= 1) {
    s1 += __shfl_xor(s1, m, kWave);
    s2 += __shfl_xor(s2, m, kWave);
  }
  if (lane == 0) {
    a.acc[ubase + j] = s1;
    a.acc2[ubase + j] = s2;
  }
}

template <int DT, int D>
void launch_rows_t(const PrefillArgs& a, hipStream_t s) {
  ProfScope ps(kProfPrefillRows, s);
  // Whole calls with output, us, one wave / four waves per row: fp32 / 64 4 units x 256 tokens 26.7 / 24.6, 2 x 512 35.0 / 29.0, 1 x 700
  // 43.1 / 31.8, 8 x 256 28.3 / 27.4, but 16 x 128 21.6 / 22.0, 30 x 128 25.3 / 27.5; fp32 / 128 8 x 256 44.1 / 37.7, 16 x 128 30.6 / 28.8;
  // bf16 / 64 4 x 256 21.4 / 20.9, 1 x 500 27.9 / 22.1, 8 x 120 16.5 / 17.4.
  const unsigned heads = static_cast<unsigned>(a.units) * a.group;
  const char* const asked = getenv("ROCO_PREFILL_WAVES_PER_ROW");
  const bool four = asked != nullptr && *asked != 0 ? asked[0] == '4' : static_cast<double>(heads) * a.L_max <= (a.L_max >= 256 || D == 128 ? 2048.0 : 1024.0) &&
                           (DT == kF32 || a.L_max > 128);
  if (four) hipLaunchKernelGGL((prefill_rows_simple<DT, D, kWaves>), dim3(a.L_max, heads), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL((prefill_rows_simple<DT, D, 1>), dim3((a.L_max + kWaves - 1) / kWaves, heads), dim3(kThreads), 0, s, a);
}

template <int DT, int D>
hipError_t launch_t(const PrefillArgs& a, hipStream_t s) {
  const dim3 grid((a.L_max + kWaves - 1) / kWaves, a.units);
  if (!a.skip_rows) launch_rows_t<DT, D>(a, s);
  {
    ProfScope ps(kProfPrefillColumns, s);
    hipLaunchKernelGGL((prefill_columns_simple<DT, D>), grid, dim3(kThreads), 0, s, a);
  }
  return hipGetLastError();
}

// The attention row of the last prompt token, P[len-1, j] for every key j, written over Acc2: the second
// statistic of the last-token importance score (section 4.1, LTAS).  One workgroup per unit; a lane group owns
// a key row, as in the passes above.  Needs the row normalisers of pass 1.
template <int DT, int D>
__global__ __launch_bounds__(kThreads) void prefill_last_row(PrefillArgs a) {
  using G = RowGeom<DT, D>;
  const int u = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / G::LPR, c = lane % G::LPR;
  const int len = a.len[u];
  const int last = len - 1;
  const size_t ubase = static_cast<size_t>(u) * a.L_max;
  const char* Kb = static_cast<const char*>(a.K) + ubase * G::ROW_BYTES;
  const int w = a.recency_window;
  const float rb = a.recency_bias_log2;
  const float inv_heads = 1.0f / static_cast<float>(a.group);
  constexpr int U = 4;  // key rows in flight per lane group: the loop is bound by load latency, not by bytes
  // the last token's query, scaled, and its normaliser: loaded once when the unit has a single head
  float q0[G::EPL];
  float lse0 = 0.0f;
  auto load_query = [&](int h, float* qs, float& lse_h) {
    const size_t qbase = (static_cast<size_t>(u) * a.group + h) * a.L_max;
    float qf[G::EPL];
    unpack16<DT>(load16(static_cast<const char*>(a.Q) + (qbase + last) * G::ROW_BYTES + c * 16), qf);
#pragma unroll
    for (int e = 0; e < G::EPL; ++e) qs[e] = qf[e] * a.scale_log2;
    lse_h = a.lse[qbase + last];
  };
  if (a.group == 1) load_query(0, q0, lse0);
  for (int base = wave * G::R; base < len; base += kWaves * G::R * U) {
    float kf[U][G::EPL];
    int jc[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int j = base + r * kWaves * G::R + g;
      jc[r] = j < len ? j : last;
      unpack16<DT>(load16(Kb + static_cast<size_t>(jc[r]) * G::ROW_BYTES + c * 16), kf[r]);
    }
    float pbar[U] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int h = 0; h < a.group; ++h) {  // the unit's query heads (one without grouped-query attention)
      float qh[G::EPL];
      float lse_h = lse0;
      if (a.group == 1) {
#pragma unroll
        for (int e = 0; e < G::EPL; ++e) qh[e] = q0[e];
      } else {
        load_query(h, qh, lse_h);
      }
#pragma unroll
      for (int r = 0; r < U; ++r) {
        float dot = 0.0f;
#pragma unroll
        for (int e = 0; e < G::EPL; ++e) dot = fmaf(qh[e], kf[r][e], dot);
        dot = group_sum<G::LPR>(dot);
        if (w > 0 && last - jc[r] < w) dot += rb;
        pbar[r] += fast_exp2(dot - lse_h);
      }
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int j = base + r * kWaves * G::R + g;
      if (c == 0 && j < len) a.acc2[ubase + j] = pbar[r] * inv_heads;
    }
  }
}

// Row normalisers handed in as natural logarithms, rescaled to the base-2 form the passes use.
__global__ __launch_bounds__(kThreads) void lse_to_base2(const float* in, float* out, size_t n) {
  const size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i < n) out[i] = in[i] * 1.4426950408889634f;
}

}  // namespace

hipError_t launch_lse_to_base2(const float* lse_ln, float* lse_log2, size_t n, hipStream_t s) {
  const size_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks == 0 || blocks > 0x7fffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(lse_to_base2, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, s, lse_ln, lse_log2, n);
  return hipGetLastError();
}

hipError_t launch_prefill_last_row(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s) {
  const dim3 grid(a.units), block(kThreads);
  if (dtype == kF32 && head_dim == 64) hipLaunchKernelGGL((prefill_last_row<kF32, 64>), grid, block, 0, s, a);
  else if (dtype == kF32 && head_dim == 128) hipLaunchKernelGGL((prefill_last_row<kF32, 128>), grid, block, 0, s, a);
  else if (dtype == kBF16 && head_dim == 64) hipLaunchKernelGGL((prefill_last_row<kBF16, 64>), grid, block, 0, s, a);
  else if (dtype == kBF16 && head_dim == 128) hipLaunchKernelGGL((prefill_last_row<kBF16, 128>), grid, block, 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

void launch_prefill_rows_simple(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s) {
  if (dtype == kBF16) launch_rows_t<kBF16, 64>(a, s);  // (bf16 / 128 has passes of its own)
  else if (head_dim == 64) launch_rows_t<kF32, 64>(a, s);
  else launch_rows_t<kF32, 128>(a, s);
}

hipError_t launch_prefill_attention_simple(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s) {
  if (dtype == kF32 && head_dim == 64) return launch_t<kF32, 64>(a, s);
  if (dtype == kF32 && head_dim == 128) return launch_t<kF32, 128>(a, s);
  if (dtype == kBF16 && head_dim == 64) return launch_t<kBF16, 64>(a, s);
  if (dtype == kBF16 && head_dim == 128) return launch_t<kBF16, 128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace roco
