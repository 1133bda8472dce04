// Instances of the general kernel for operands whose rows are too far apart for offsets in 32 bits
// (general_offsets_fit): the same tiles with a 64-bit address per lane and chunk.
// Measured against the 64 x 64 kernel for short runs, which shifts every chunk and took all rows from 32 MiB apart on (us): bf16 TN
// 40,000,000 x 64 x 64 5100 -> 3614, 40,000,003 x 128 x 200 15290 -> 8442, NN 64 x 40,000,000 x 64 5428 -> 4965, fp32 TN 40,000,000 x 32 x 48
// 6992 -> 5497, int8 x 64 x 128 5423 -> 4774; bf16 NT 128 x 2000 x 4096 with A's rows 76 MiB apart 42.5 -> 10.8.  Rows that do fit, by what a tile
// spans and not by the pitch: bf16 TN 20,000,000 x 64 x 64 2524 -> 1725, NT 1 x 16 x 2^24 11490 -> 1478.
#include "general.hpp"

namespace brg {

hipError_t general_launch_far(const Problem &p, int tile)
{
    if (p.A_off)
        return general_launch_far_offsets(p, tile);
    if (p.in_s8)
        return general_layout<KIND_S8, false, ROWS_FAR>(p, tile);
    if (p.in_f8)
        return p.f8_e5m2 ? general_layout<KIND_BF8, false, ROWS_FAR>(p, tile) : general_layout<KIND_F8, false, ROWS_FAR>(p, tile);
    if (in_16bit(p))
        return p.in_f16 ? general_layout<KIND_F16, false, ROWS_FAR>(p, tile) : general_layout<KIND_BF16, false, ROWS_FAR>(p, tile);
    return general_layout<KIND_F32, false, ROWS_FAR>(p, tile);
}

}  // namespace brg
