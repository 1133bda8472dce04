// Instances of the 256 x 256 x 64 ping-pong kernel for a K that is no multiple of 64.
#include "bf16_pingpong.hpp"

namespace brg {

hipError_t launch_pingpong_tail(const Problem &p)
{
    void (*kern)(Bf16Args) = nullptr;
    if (p.in_f16)
        BRG_PP_PICK(kern, p, KIND_F16, false, true);
    else
        BRG_PP_PICK(kern, p, KIND_BF16, false, true);
    return pingpong_launch(kern, p);
}

}  // namespace brg
