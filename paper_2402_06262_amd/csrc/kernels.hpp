// Internal launch interface between the C ABI (api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace roco {

// Eviction policy in the paper's two-stage framework (section 4): an eviction scope, then an importance score
// inside it.  All zeros is RoCo (section 4.3).
enum : int { kImpMas = 0, kImpAas = 1, kImpOldest = 2, kImpLast = 3, kImpCount = 4 };
enum : int { kScopeStd = 0, kScopeWindow = 1, kScopeAll = 2 };
struct Policy {
  int importance;  // kImpMas: Acc/Count; kImpAas: Acc; kImpOldest: position, the first `sinks` positions last;
                   // kImpLast: the attention from the latest query, kept in the second statistics plane;
                   // kImpCount: how many queries gave the token more than their row's average attention, ditto
  int scope_kind;  // kScopeStd: lowest variance; kScopeWindow: lowest position (oldest); kScopeAll: everything
  int sinks;
  // the second plane holds the latest query's probability instead of the accumulated squares
  __host__ __device__ bool keeps_last_score() const { return importance == kImpLast; }
  // ... or counts the queries whose probability for the token was above 1 / (tokens the query attended)
  __host__ __device__ bool counts_above_average() const { return importance == kImpCount; }
  // The second statistic after a query that attended `attended` tokens gave the token probability p.
  __host__ __device__ float second_statistic(float old, float p, float attended) const {
    if (importance == kImpLast) return p;
    if (importance == kImpCount) return old + (p * attended > 1.0f ? 1.0f : 0.0f);
    return old + p * p;
  }
  // its keys are probabilities or sums of them, not positions or counts
  __host__ __device__ bool spreads_importance() const { return importance != kImpOldest && importance != kImpCount; }
  __host__ __device__ bool scope_is_window() const { return scope_kind == kScopeWindow; }  // its keys are positions
  __host__ __device__ bool needs_pos() const { return importance == kImpOldest || scope_kind == kScopeWindow; }
  // number of tokens inside the scope when n are cached
  __host__ __device__ int scope_size(int scope, int n) const { return scope_kind == kScopeAll ? n : scope; }
};

constexpr int kMaxSplits = 64;        // upper bound on split-K partials per unit (sizes the workspace)
constexpr int kDecodeSelectThreads = 256;
constexpr int kMaxFusedBudget = 4096;       // largest budget of the one-kernel decode step (keys and logits in LDS)
constexpr int kMaxDecodeBudgetLds = 16384;  // ranking keys of a unit are kept in LDS up to here (128 KiB), else in the workspace
constexpr size_t kDefaultDynamicLds = 65536;  // LDS a kernel may use without raising its limit first
constexpr size_t kStaticLdsAllowance = 16384;  // upper bound on the statically declared LDS of the kernels that ask

// Dynamic LDS for the ranking keys of one unit (0: they go to the workspace); raises the kernel's limit when the
// request, together with what the kernel declares statically, may be above the default one -- to the most that any call asks for,
// since another thread's smaller call might lower it again before the launch.  Returns false if the runtime refuses.
inline size_t key_lds_bytes(int B) {
  return B <= kMaxDecodeBudgetLds ? static_cast<size_t>(B) * 2 * sizeof(uint32_t) : 0;
}
inline bool allow_key_lds(const void* kernel, size_t bytes) {
  constexpr size_t kMost = static_cast<size_t>(kMaxDecodeBudgetLds) * 2 * sizeof(uint32_t);
  if (bytes + kStaticLdsAllowance <= kDefaultDynamicLds) return true;
  return bytes <= kMost && hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMost)) == hipSuccess;
}

struct DecodeArgs {
  int units, B, scope, splits, rows_per_split;
  Policy pol;
  int unroll;            // rows in flight per lane group in decode_attend: 2, 4 or 8
  int fused;             // 1: one workgroup does the whole step of a unit (decode_fused), no workspace traffic
  int streaming;         // 1: K / V rows are loaded with the non-temporal hint (cache far larger than the last-level cache)
  int rotate;            // stagger the start offset of every workgroup inside its slot range
  float scale_log2;      // scale * log2(e)
  int recency_window;
  float recency_bias_log2;
  const void *q, *k_new, *v_new;
  const int32_t* qpos;
  void *K, *V;
  float* stats;          // [units][3][B]
  int32_t *pos, *n_used;
  int32_t* next_slot;    // [units] victim chosen for the next step (valid while the unit is full)
  void* out;
  int32_t *evicted_slot, *evicted_pos;
  // workspace
  float* z;              // [units][B]   base-2 logits of this step
  float* part_m;         // [units][splits]
  float* part_l;         // [units][splits]
  float* part_o;         // [units][splits][D]
  uint32_t* keys;        // [units][2][B] ranking keys when B is too large for LDS, else unused
};

constexpr int kMaxKeyShares = 4;     // PrefillArgs::ksplit
constexpr int kMaxQueryShares = 16;  // PrefillArgs::qsplit

struct PrefillArgs {
  int units, L_max, B, scope;
  int group;             // query heads per unit (1 without grouped-query attention): Q and lse are [units][group][L_max]
  Policy pol;
  int pairs;             // matrix-core path: workgroup ids per unit (set by its launcher)
  int whole;             // ... and the units whose workgroups all go to one die (ditto; see locate)
  int paired;            // matrix-core path: 1 = long+short block per workgroup, 0 = one block, -1 = choose
  int skip_rows;         // 1: lse already holds the row normalisers, pass 1 is not run
  int qsplit;            // matrix-core path: workgroups that share a block of keys, each with a part of the queries (set by its launcher)
  int ksplit;            // matrix-core path, row pass: workgroups that share a block of queries (ditto)
  int shares;            // pairs of planes for column sums that the workspace has, 2 at least
  int row_bytes;         // of K and V, for the selection (set by its launcher)
  int shares_to_add;     // > 1: the column sums lie in that many shares, which the selection adds (set by the passes' launcher)
  float scale_log2;
  int recency_window;
  float recency_bias_log2;
  const void *Q, *K, *V;
  const int32_t* len;
  void *K_cache, *V_cache;
  float* stats;          // [units][3][B]
  int32_t *pos, *n_used;
  int32_t* next_slot;    // [units]
  void* O;               // may be null
  // workspace
  const float* lse_given;  // roco_prefill_compress_lse: the caller's natural log-sum-exps until they have been rescaled to `lse`, else null
  float lse_scale;         // what the column pass multiplies the normalisers by as it reads them: 1, or log2(e) for lse_given
  float* lse;            // [units][group][L_max]  base-2 log-sum-exp of every query row
  float* acc;            // [units][L_max]; acc, acc2, var_key, mas_key and what follows are planes of `plane` words side by side
  float* acc2;           // [units][L_max]
  uint32_t* var_key;     // [units][L_max]
  uint32_t* mas_key;     // [units][L_max]
  size_t plane;
  // where share `share` of a pass that several workgroups divide leaves its sums (which = 0: Acc, 1: Acc2): the first in acc and
  // acc2, the second in the planes that the selection will later use for its ranking keys, further ones behind those
  __host__ __device__ float* sums_of(int share, int which) const { return acc + static_cast<size_t>(2 * share + which) * plane; }
  // ... and its row normalisers: the first where they belong, the others in the planes of the column sums, all heads together:
  // from the first plane on if they are merged before the column pass, behind the planes that it writes if it merges them itself
  // as it reads them (lse_shares > 1; see columns_merge_normalisers)
  int lse_shares, lse_behind;
  __host__ __device__ float* lse_of_share(int share) const {
    return share == 0 ? lse : acc + lse_behind * plane + static_cast<size_t>(share - 1) * units * group * L_max;
  }
  // most shares whose normalisers have room there
  int row_shares() const {
    const size_t room = 1 + 2 * static_cast<size_t>(shares) * plane / (static_cast<size_t>(units) * group * L_max);
    return room < kMaxKeyShares ? static_cast<int>(room) : kMaxKeyShares;
  }
};

constexpr int kMaxBlock = 64;        // query rows (tokens x heads) per block-wise step: two 32-wide matrix tiles
constexpr int kBlockPartials = 8 * kMaxBlock;  // split-K partials per unit of the block-wise step: splits times rows of the planes
constexpr int kMaxSplitRows = 1 << 22;  // slots of a split of the block-wise step: 2^30 bytes of a bf16 / 128 operand

struct BlockArgs {
  int units, B, scope, block, splits, rows_per_split;
  Policy pol;
  int streaming;  // as DecodeArgs::streaming
  int row_bytes;  // bytes of a K / V / q row
  int single;     // 1: single-token step without block_prepare (set by launch_block)
  int heads;    // query heads that share the unit's keys and values (1 without grouped-query attention)
  int queries;  // query rows per unit = block * heads <= 64; row r belongs to token r / heads, head r % heads
  int qrows;    // rows per unit of the z / part_* planes, a power of two: 32 or 64 (bf16 / 128), else 8 to 64
  float scale_log2;
  int recency_window;
  float recency_bias_log2;
  const void *q, *k_new, *v_new;   // q [units][block][heads][128], k_new / v_new [units][block][128] bf16
  const int32_t* qpos0;            // [units]
  void *K, *V;
  float* stats;
  int32_t *pos, *n_used, *next_slot;
  void* out;                       // [units][block][heads][128] bf16
  int32_t *evicted_slot, *evicted_pos;  // [units][block], may be null
  // workspace
  int32_t* blk_idx;                // [units][B]   block token index held by a slot, -1 for older tokens
  float* z;                        // [units][qrows][B] base-2 logits
  float* part_m;                   // [units][splits][qrows]
  float* part_l;                   // [units][splits][qrows]
  float* part_o;                   // [units][splits][qrows][128]
  uint32_t* keys;                  // [units][2][B] when B is too large for LDS
};
hipError_t launch_block(int dtype, int head_dim, const BlockArgs& a, hipStream_t s);  // B % 4 == 0
// The step of bf16 in one or two kernels, if that is the quicker way (BlockArgs::single is set); else false and nothing is launched.
bool launch_block_fused(int head_dim, const BlockArgs& a, hipStream_t s, hipError_t& e);

// dtype: 0 = f32, 1 = bf16; head_dim: 64 or 128.  Each returns hipGetLastError() of its launches.
hipError_t launch_decode(int dtype, int head_dim, const DecodeArgs& a, hipStream_t s);
int decode_rows_per_pass(int dtype, int head_dim, int unroll);  // granularity of DecodeArgs::rows_per_split
hipError_t launch_cache_read_probe(int dtype, int head_dim, const DecodeArgs& a, hipStream_t s);
hipError_t launch_mfma_probe(int workgroups, int iters, int mode, float* sink, hipStream_t s);  // mode: ROCO_PROBE_*
hipError_t launch_select_victims(const DecodeArgs& a, hipStream_t s);
// uses stats, pos, n_used, keys; writes mask[units][B] (1 = survives a shrink of the unit to `keep` tokens)
hipError_t launch_select_retained(const DecodeArgs& a, int keep, int32_t* mask, hipStream_t s);  // uses stats, n_used, next_slot, keys
// |A and B| and |A or B| per unit of two sets of cached positions in [0, max_pos), max_pos <= 524288
hipError_t launch_set_overlap(int units, int slots_a, const int32_t* pos_a, const int32_t* mask_a, const int32_t* n_a,
                              int slots_b, const int32_t* pos_b, const int32_t* mask_b, const int32_t* n_b, int max_pos,
                              int32_t* inter, int32_t* uni, hipStream_t s);
hipError_t launch_prefill_attention_simple(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s);
// The matrix-core passes: bf16 / 128, and the other forms.  Both may leave PrefillArgs::shares_to_add set for prefill_select.
hipError_t launch_prefill_attention_mfma(PrefillArgs& a, hipStream_t s);
hipError_t launch_prefill_attention_planes(int dtype, int head_dim, PrefillArgs& a, hipStream_t s);
struct PassPlan;  // prefill_schedule.hpp
void launch_prefill_rows_planes_wide(const PrefillArgs& a, const PassPlan& plan, hipStream_t s);
void launch_prefill_columns_planes_wide(PrefillArgs& a, const PassPlan& plan, hipStream_t s);
// Prompts of few scores: the vector-ALU row pass, one wave per query and as many waves as queries, is done before a
// workgroup of the matrix-core pass has walked its tiles one after the other.  Row pass, us, vector against matrix:
//   fp32 / 64 with output (2^19 scores)   4 units x 256 tokens 12.5 / 18.9, 2 x 512 19.6 / 28.6, 16 x 128 10.2 / 14.3, but
//                                         32 x 128 15.0 / 14.2 and 128 x 64 16.6 / 16.1
//   fp32 / 128 with output (2^19)         8 x 256 24.5 / 38.0, 32 x 128 23.6 / 25.3, but 128 x 64 26.0 / 25.3
//   bf16 / 64 with output (2^18)          4 x 256 10.8 / 12.5, 2 x 362 13.2 / 14.5, 16 x 128 9.5 / 10.3, but 64 x 64 9.8 / 8.9
//   fp32 / 64 without (192 tokens, 2^17)  8 x 128 8.8 / 9.2, 4 x 150 9.7 / 10.9, 2 x 160 9.4 / 10.2, but 1 x 200 10.5 / 10.6
//   fp32 / 128 without (128 tokens, 2^17) 8 x 128 12.8 / 14.6, 13 x 100 12.5 / 14.5, but 1 x 140 13.2 / 12.4 and 4 x 150
//                                         15.0 / 13.5
inline bool prefill_is_tiny(const PrefillArgs& a, double scores) {
  return static_cast<double>(a.units) * a.group * a.L_max * a.L_max <= scores;
}
inline bool prefill_rows_are_tiny(const PrefillArgs& a, bool fp32, int head_dim) {
  if (a.O != nullptr) return prefill_is_tiny(a, fp32 ? 524288.0 : 262144.0);
  return fp32 && a.L_max <= (head_dim == 64 ? 192 : 128) && prefill_is_tiny(a, 131072.0);
}
void launch_prefill_rows_simple(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s);  // the row pass alone
// the shares of PrefillArgs::ksplit / qsplit merged into the first ones
void launch_merge_key_shares(const PrefillArgs& a, hipStream_t s);
// The selection adds the shares of the column sums itself where it keeps its ranking keys in LDS, not in the planes of the
// second share, and nothing else comes between; else, and for more than two shares of more than 2048 tokens, a kernel of its
// own does: 3 to 5 us of a call, which one workgroup per unit takes too for four shares of 4096 tokens (2 x 6872: selection 30
// us with two shares, 36 with eight, 41 with sixteen), but not for a few hundred.
inline bool selection_adds_shares(const PrefillArgs& a, int shares) {
  return (shares <= 2 || a.L_max <= 2048) && a.L_max <= kMaxDecodeBudgetLds && !a.pol.keeps_last_score();
}
void join_query_shares(PrefillArgs& a, const PrefillArgs& pass, hipStream_t s);
// overwrites PrefillArgs::acc2 with the attention row of each unit's last prompt token (kImpLast)
hipError_t launch_lse_to_base2(const float* lse_ln, float* lse_log2, size_t n, hipStream_t s);
// writes PrefillArgs::lse from lse_given, if there is one left to rescale (one launch); false if the launch fails
inline bool rescale_given_lse(PrefillArgs& a, hipStream_t s) {
  if (a.lse_given == nullptr) return true;
  const float* const given = a.lse_given;
  a.lse_given = nullptr;
  return launch_lse_to_base2(given, a.lse, static_cast<size_t>(a.units) * a.group * a.L_max, s) == hipSuccess;
}
hipError_t launch_prefill_last_row(int dtype, int head_dim, const PrefillArgs& a, hipStream_t s);
hipError_t launch_prefill_select_compact(int dtype, int head_dim, PrefillArgs a, hipStream_t s);

}  // namespace roco
