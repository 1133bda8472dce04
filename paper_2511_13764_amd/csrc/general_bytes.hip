// Instances of the general kernel for one-byte operands: int8 on the integer matrix
// instruction (exact), FP8 E4M3 / E5M2 widened to bf16 on the way into LDS, so that their
// products are exact and their sums fp32 (the 128-deep FP8 instruction would cut them).
#include "general.hpp"

namespace brg {

hipError_t general_launch_bytes(const Problem &p, int tile)
{
    if (p.in_s8)
        return general_layout<KIND_S8, false>(p, tile);
    return p.f8_e5m2 ? general_layout<KIND_BF8, false>(p, tile) : general_layout<KIND_F8, false>(p, tile);
}

}  // namespace brg
