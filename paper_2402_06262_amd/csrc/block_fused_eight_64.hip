// Shapes of block_fused.hpp for bf16 / 64 with eight waves: 16 query rows.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch<64, 8, 1, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch<64, 8, 1, 8>(const BlockArgs&, hipStream_t);
template hipError_t launch<64, 8, 1, 16>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
