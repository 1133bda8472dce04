// Instances of the general kernel for 16-bit operands (bf16, binary16; packed B included).
#include "general.hpp"

namespace brg {

hipError_t general_launch_half(const Problem &p, int tile)
{
    return p.in_f16 ? general_layout<KIND_F16, false>(p, tile) : general_layout<KIND_BF16, false>(p, tile);
}

}  // namespace brg
