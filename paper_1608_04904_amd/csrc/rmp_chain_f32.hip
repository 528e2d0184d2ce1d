// Instances of the MD chain with FP32 state.
#include "rmp_chain.h"

namespace rmp {
RMP_CHAIN_SHAPES(RMP_CHAIN_DEF, float)
}  // namespace rmp
