// The same for batch-reduce calls whose tiles are given by offset lists.
#include "general.hpp"

namespace brg {

hipError_t general_launch_far_offsets(const Problem &p, int tile)
{
    if (p.in_f16)
        return general_layout<KIND_F16, true, ROWS_FAR>(p, tile);
    return p.in_bf16 ? general_layout<KIND_BF16, true, ROWS_FAR>(p, tile) : general_layout<KIND_F32, true, ROWS_FAR>(p, tile);
}

}  // namespace brg
