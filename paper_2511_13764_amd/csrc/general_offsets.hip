// Instances of the general kernel for batch-reduce calls whose tiles are given by offset
// lists (16-bit and fp32 operands).
#include "general.hpp"

namespace brg {

hipError_t general_launch_offsets(const Problem &p, int tile)
{
    if (p.in_f16)
        return general_layout<KIND_F16, true>(p, tile);
    return p.in_bf16 ? general_layout<KIND_BF16, true>(p, tile) : general_layout<KIND_F32, true>(p, tile);
}

}  // namespace brg
