// Shapes of block_fused.hpp for bf16 / 128 with four waves: 17 to 32 query rows.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch<128, 4, 2, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch<128, 4, 2, 8>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
