// Shapes of block_fused.hpp for bf16 / 64 with 33 to 64 query rows, half of the tokens in each of two workgroups.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch_halves<64, 8, 2, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch_halves<64, 8, 2, 8>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
