// Shapes of block_fused.hpp for bf16 / 64 with eight waves: 17 to 32 query rows.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch<64, 8, 2, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch<64, 8, 2, 8>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
