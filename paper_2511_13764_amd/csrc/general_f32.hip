// Instances of the general kernel for fp32 operands.
#include "general.hpp"

namespace brg {

hipError_t general_launch_f32(const Problem &p, int tile) { return general_layout<KIND_F32, false>(p, tile); }

}  // namespace brg
