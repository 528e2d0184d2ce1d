// Instances of the MD chain with FP64 state.
#include "rmp_chain.h"

namespace rmp {
RMP_CHAIN_SHAPES(RMP_CHAIN_DEF, double)
}  // namespace rmp
