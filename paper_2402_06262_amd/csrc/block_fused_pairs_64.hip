// Shapes of block_fused.hpp for bf16 / 64 with four waves, of which a compute unit holds two workgroups: 16 query rows.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch<64, 4, 1, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch<64, 4, 1, 8>(const BlockArgs&, hipStream_t);
template hipError_t launch<64, 4, 1, 16>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
