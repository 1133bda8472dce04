// Instances of the 128-row streaming kernel for a K that is no multiple of 64, in its three tiles.
#include "bf16_stream128.hpp"

namespace brg {

namespace {

template <int KIND, int BN>
hipError_t launch(const Problem &p)
{
    const bool ak = p.transA == 0;
    void (*kern)(Bf16Args) =
        p.b_packed ? (ak ? bf16_stream128_kernel<true, LAY_PACKED, KIND, BN, true> : bf16_stream128_kernel<false, LAY_PACKED, KIND, BN, true>)
        : p.transB ? (ak ? bf16_stream128_kernel<true, LAY_K, KIND, BN, true> : bf16_stream128_kernel<false, LAY_K, KIND, BN, true>)
                   : (ak ? bf16_stream128_kernel<true, LAY_MN, KIND, BN, true> : bf16_stream128_kernel<false, LAY_MN, KIND, BN, true>);
    return stream128_launch<BN>(kern, p);
}

template <int KIND>
hipError_t launch_tile(const Problem &p, TailKernel k)
{
    switch (k) {
    case TAIL_NARROW: return stream128_launch<48>(bf16_stream128_kernel<true, LAY_K, KIND, 48, true>, p);
    case TAIL_128: return launch<KIND, 128>(p);
    case TAIL_WIDE: return launch<KIND, 256>(p);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_stream_tail(const Problem &p, TailKernel k)
{
    return p.in_f16 ? launch_tile<KIND_F16>(p, k) : launch_tile<KIND_BF16>(p, k);
}

}  // namespace brg
