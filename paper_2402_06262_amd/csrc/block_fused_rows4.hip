// The shapes of block_fused.hpp for 17 to 32 query rows, four waves.
#include "block_fused.hpp"

namespace roco {
namespace fused {
template hipError_t launch<4, 2, 4>(const BlockArgs&, hipStream_t);
template hipError_t launch<4, 2, 8>(const BlockArgs&, hipStream_t);
}  // namespace fused
}  // namespace roco
