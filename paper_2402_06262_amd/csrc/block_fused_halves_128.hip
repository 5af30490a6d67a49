// Shapes of block_fused.hpp for bf16 / 128 with half of the tokens in each of two workgroups: 33 to 64 query rows, and 25 to 32 over more than 1024 slots.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch_halves<128, 4, 1, 16>(const BlockArgs&, hipStream_t);
template hipError_t launch_halves<128, 8, 2, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch_halves<128, 8, 2, 8>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
