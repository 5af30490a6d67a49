// When the one-kernel step of block_fused.hpp is taken, and in which shape.
#include <cstdlib>

#include "block_fused.hpp"

namespace roco {
namespace fused {

extern template hipError_t launch<128, 4, 1, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 4, 1, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 4, 1, 16>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 8, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 8, 2, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 4, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 4, 2, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 8, 1, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 8, 1, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<128, 8, 1, 16>(const BlockArgs&, hipStream_t);
extern template hipError_t launch_halves<128, 4, 1, 16>(const BlockArgs&, hipStream_t);
extern template hipError_t launch_halves<128, 8, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch_halves<128, 8, 2, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 4, 1, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 4, 1, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 4, 1, 16>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 8, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 8, 2, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 4, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 4, 2, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 8, 1, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 8, 1, 8>(const BlockArgs&, hipStream_t);
extern template hipError_t launch<64, 8, 1, 16>(const BlockArgs&, hipStream_t);
extern template hipError_t launch_halves<64, 8, 2, 4>(const BlockArgs&, hipStream_t);
extern template hipError_t launch_halves<64, 8, 2, 8>(const BlockArgs&, hipStream_t);

using Launch = hipError_t (*)(const BlockArgs&, hipStream_t);

// Splits belong to the three kernels: whoever asks for a number of them gets those (0 asks for none).
static bool asks_for_splits() {
  const char* const e = getenv("ROCO_BLOCK_SPLITS");
  return e != nullptr && atoi(e) > 0;
}

// The shape for W waves: the fewest tiles per wave that hold the unit's slots, null if none does.
template <int HD, int W, int NQ, int ZT, int... MORE>
Launch shape_for(const BlockArgs& a) {
  if (Shape<HD, W, NQ, ZT>::takes(a)) return launch<HD, W, NQ, ZT>;
  if constexpr (sizeof...(MORE) > 0) return shape_for<HD, W, NQ, MORE...>(a);
  return nullptr;
}

// 33 to 64 rows: each half of the tokens in a workgroup of its own, where the pairs take one round and the stream, which both read,
// is long enough.  Against the three kernels, us per step, bf16 / 128: 128 units x 2048 slots x 16 tokens of 4 heads 95 / 65, 48 x 1024
// x 16 of 4 53 / 37, 4 x 476 x 48 39.9 / 34.1, 7 x 1804 x 19 of 2 48.0 / 46.6.  Two rounds, above 768 slots: 256 x 1300 x 16 of 4 107 / 80,
// 130 x 2048 x 32 of 2 103.1 / 103.0, 256 x 2048 x 32 of 2 136 / 130; tokens of one head have twice the sums to add, and the three kernels
// fill their rounds badly with the three splits that 171 to 240 units get (180 x 2048 x 33 105 / 95, 220 x 1536 x 64 123 / 103) but well
// beside them (150 x 1536 x 48 86 / 90, 161 x 1100 x 64 88 / 91, 256 x 780 x 33 60.6 / 65.6, 256 x 2048 x 64 138 / 143; 256 x 2048 x 17
// of 2 111 / 115); up to 768 slots 176 x 584 x 41 66 / 68, 140 x 248 x 46 53 / 57; more rounds: 512 x 1536 x 10 of 4 166 / 175, 423 x 244
// x 61 77 / 125.
// bf16 / 64, whose three kernels do not use the matrix cores: 128 x 96 x 48 39.2 / 27.5, 180 x 132 x 33 52.9 / 43.7, 256 x 160 x 64 66.3 /
// 56.6, 256 x 96 x 12 of 4 39.2 / 34.0, 400 x 260 x 64 126 / 108, 800 x 224 x 33 146 / 139; but where their workgroups of 64 slots are
// resident at once and the pairs are not 180 x 64 x 48 36.9 / 47.9, 256 x 128 x 33 39.9 / 40.9, 155 x 168 x 56 49.3 / 53.6; and 878 x 144 x 46
// 133 / 151, 758 x 104 x 46 95 / 124.
template <int HD>
Launch choose_halves(const BlockArgs& a) {
  const BlockArgs half = half_step(a);
  if (a.block < 2 || a.pol.keeps_last_score() || a.pol.counts_above_average()) return nullptr;
  const Launch two = Shape<HD, 8, 2, 4>::takes(half)   ? launch_halves<HD, 8, 2, 4>
                     : Shape<HD, 8, 2, 8>::takes(half) ? launch_halves<HD, 8, 2, 8>
                                                       : nullptr;
  const char* const asked = getenv("ROCO_BLOCK_FUSED");
  if (asked != nullptr && *asked != 0) return asked[0] == '0' ? nullptr : two;
  if (two == nullptr || asks_for_splits()) return nullptr;
  if (HD == 64) {
    const bool resident = a.units * ((a.B + 63) / 64) <= 512;  // the three kernels' workgroups
    return a.units <= 128 || (a.units <= 256 && (!resident || a.heads >= 4)) || a.B >= 224 ? two : nullptr;
  }
  const bool two_rounds = a.heads >= 4 || (a.heads > 1 && a.queries > 48) || (a.units > 170 && a.units < 240);
  return a.units <= 128 || (a.units <= 256 && a.B > 768 && two_rounds) ? two : nullptr;
}

// Up to 32 rows.  One workgroup per unit needs units enough, or caches so small that the launches it saves count for more.  Against the
// three kernels, us per step, bf16 / 128:
//   up to 16 rows, B <= 1024: always (1 unit x 120 slots x 16 heads 13.7 / 9.2, 4 x 368 x 16 tokens 26.4 / 22.7, 20 x 944 x 2 heads
//   17.6 / 16.7, 161 x 228 x 16 heads 25.1 / 13.8); B <= 2048 from 72 units on (48 x 1536 x 4 heads 25.0 / 28.1, 64 x 2048 x 4 heads
//   32.6 / 34.6, 80 x 1536 x 4 heads 30.7 / 29.9, 128 x 2048 x 4 heads 45.9 / 38.4), B <= 4096 from 80 on (64 x 3072 x 4 heads
//   41.3 / 48.2, 80 x 3072 55.6 / 50.1, 192 x 4096 117 / 76).
//   17 to 32 rows, B <= 1024: always (1 x 892 x 21 tokens 32.1 / 32.0, 511 x 132 x 20 rows 45.9 / 27.8); B <= 2048 from 65 units on (62 x
//   2044 x 28 rows 53.0 / 54.6, 65 x 2048 x 6 of 4 58.4 / 53.1, 140 x 1712 x 32 85 / 72, 256 x 2048 x 32 108 / 85, 447 x 2048 x 5 of 4 156 / 131).
//   Above 24 rows, where eight waves' workgroups do not fill a round or do not fit it, half of the tokens in each of two workgroups of
//   four waves (three kernels / eight waves / halves): 65 x 2048 x 32 69 / 70 / 60, 97 x 1628 x 32 74 / 67 / 57, 264 x 1536 x 32 115 / 123 /
//   109, 512 x 2048 x 32 184 / 170 / 168, 697 x 1792 x 32 264 / 231 / 220; but 140 x 1352 x 6 of 4 66 / 49 / 54, 400 x 1960 x 17 143 / 132 / 144.
// bf16 / 64, half of the bytes: B <= 2048 always (10 units x 1508 slots x 4 heads 19.0 / 17.0, 1 x 1800 x 24 tokens 44.0 / 42.7, 171 x 992 x
//   16 heads 47.0 / 16.5, 518 x 1904 x 20 rows 308 / 144), but for more than 24 rows of more than 1536 slots on few units (1 x 2048 x 32 48.7 / 52.4, 12 x 1800 x 32 51.5 /
//   52.2, 24 x 2048 x 32 56.8 / 53.5).  B <= 4096 from 40 units on (24 x 4096 x 4 heads 31.1 / 33.5, 32 x 3000 x 4 tokens 39.2 / 39.7,
//   44 x 3000 x 4 heads 34.2 / 29.4, 44 x 2052 x 4 tokens 36.5 / 34.4, 110 x 4096 x 8 heads 73.2 / 36.9), of single tokens of 8 and more
//   heads from 24 on (24 x 3000 x 8 29.6 / 29.0, x 16 37.1 / 29.5).  A recency window, whose bias is one workgroup's work here, moves
//   these lines (4 x 1024 x 2 heads 16.1 / 13.8, but 4 x 2048 x 2 heads 20.0 / 21.6, 4 x 2048 x 24 tokens 47.3 / 49.5, 32 x 2048 x 2 heads
//   21.4 / 22.1, 44 x 2052 x 2 25.4 / 27.3, 32 x 3000 x 8 30.8 / 33.4).
// Four waves, two workgroups to a compute unit, where the units are more than the compute units (512 x 16 tokens x 2048 with eight
// 119.7, with four 110.8; 356 x 2 heads x 132 23.0 / 14.1) and where a cache is a tile or two per wave (1 x 120 x 16 heads 10.1 / 9.2),
// else eight (256 x 16 tokens x 2048 58.7 / 67.8, 128 x 4 heads x 2048 38.4 / 43.0).
// ROCO_BLOCK_FUSED=8, 4, 2, 0: eight waves, four, halves, three kernels (tests run all); a shape that does not take the step leaves it to
// the three kernels.
template <int HD>
Launch choose(const BlockArgs& a) {
  if (a.queries > 2 * kQ16) return choose_halves<HD>(a);
  const bool one = a.queries <= kQ16;
  const Launch eight = one ? shape_for<HD, 8, 1, 4, 8, 16>(a) : shape_for<HD, 8, 2, 4, 8>(a);
  const Launch four = one ? shape_for<HD, 4, 1, 4, 8, 16>(a) : shape_for<HD, 4, 2, 4, 8>(a);
  const char* const asked = getenv("ROCO_BLOCK_FUSED");
  Launch halves = nullptr;
  if constexpr (HD == 128) {
    if (!one && a.block > 1 && !a.pol.keeps_last_score() && !a.pol.counts_above_average() && Shape<HD, 4, 1, 16>::takes(half_step(a)))
      halves = launch_halves<HD, 4, 1, 16>;
  }
  if (asked != nullptr && *asked != 0) return asked[0] == '2' ? halves : asked[0] == '8' ? eight : asked[0] == '4' ? four : nullptr;
  if (asks_for_splits()) return nullptr;
  const bool pairs = four != nullptr && (a.units > 256 || a.B <= 256);
  if (halves != nullptr && a.B > 1024 && a.queries > 24 && (a.units > 256 || (a.units > 64 && a.units <= 128))) return halves;
  int least = 0;
  if (HD == 64) {
    const bool window = a.recency_window > 0, wide = a.block == 1 && a.queries >= 8;
    if (a.B > 2048) least = window ? (wide ? 40 : 60) : wide ? 24 : 40;
    else if (a.B > 1536) least = window ? 40 : a.queries > 24 ? 24 : 0;
  } else if (a.B > 1024) {
    least = a.B <= 2048 ? (one ? 72 : 65) : 80;
  }
  if (a.units < least || (HD == 128 && !pairs && a.queries > 24 && a.units > 256)) return nullptr;
  return pairs ? four : eight;
}

}  // namespace fused

bool launch_block_fused(int head_dim, const BlockArgs& a, hipStream_t s, hipError_t& e) {
  const fused::Launch step = head_dim == 128 ? fused::choose<128>(a) : fused::choose<64>(a);
  if (step == nullptr) return false;
  ProfScope ps(kProfBlockAttend, s);
  e = step(a, s);
  return true;
}

}  // namespace roco
