// The 64 x 64 and 128 x 64 tiles of the streaming kernel with its waves divided by kind (bf16_stream128.hpp): four waves
// multiply, four load, a ring of four blocks of 16 KiB or three of 24.
//
// What they are for: grids that 128 x 128 tiles leave most of the CUs idle on, where a split of the reduction costs a
// second launch and its partial sums (4 to 6 us), and 32 x 128 tiles pull more bytes per flop.
// What bounds them: what a CU pulls from the caches, 16 KiB per 0.20 us (82 B/ns), 24 KiB per 0.27, after 3.7 us for a launch of one block.  Counters of
// 1024^3: 67 MB of requests, which L2 serves at up to 125 B/ns and CU (2.1 us), 12.9 MB of them from beyond it (1.8 us at the 7.1 TB/s that all CUs get there);
// no bank conflict but the 64 a workgroup has in its epilogue, in any layout.  The general
// kernel's divided tiles, which took the same blocks through registers, 5 to 10 % more.  A deeper ring changes nothing (8 blocks of 16 KiB
// cost the second workgroup: 2048 x 1024 x 1024 10.2 -> 14.3 us).
// Measured, plan before -> now (us): 1024^3 NN 9.0 -> 7.9, NT 9.3 -> 7.6, 696 x 1024 x 2816 NT (32 x 128 tiles) 18.4 -> 13.1, 320 x 1792 x 2112 TN
// (128 x 128, split 5) 15.7 -> 11.2; 128 x 64: 2048 x 1024 x 1024 TN 13.3 -> 10.4, 512 x 4096 x 4096 NT (128 x 128, split 2) 26.1 -> 24.1.
#include "bf16_stream128.hpp"

namespace brg {

namespace {

template <int KIND, int BM, bool TOTAL>
hipError_t launch(const Problem &p)
{
    const bool ak = p.transA == 0;
    void (*kern)(Bf16Args) =
        p.b_packed ? (ak ? bf16_stream128_kernel<true, LAY_PACKED, KIND, 64, false, BM, TOTAL> : bf16_stream128_kernel<false, LAY_PACKED, KIND, 64, false, BM, TOTAL>)
        : p.transB ? (ak ? bf16_stream128_kernel<true, LAY_K, KIND, 64, false, BM, TOTAL> : bf16_stream128_kernel<false, LAY_K, KIND, 64, false, BM, TOTAL>)
                   : (ak ? bf16_stream128_kernel<true, LAY_MN, KIND, 64, false, BM, TOTAL> : bf16_stream128_kernel<false, LAY_MN, KIND, 64, false, BM, TOTAL>);
    return stream128_launch<64, BM>(kern, p);
}

// (128 x 64 has registers for two workgroups on a CU without the totals only)
template <int KIND>
hipError_t launch_tile(const Problem &p, int tile)
{
    if (tile == GEN_64)
        return launch<KIND, 64, true>(p);
    return p.c_f32 || p.split > 1 ? launch<KIND, 128, true>(p) : launch<KIND, 128, false>(p);
}

}  // namespace

bool stream_form_runs(const Problem &p, int tile)
{
    return (tile == GEN_64 || tile == GEN_MID) && p.batch == 1 && !p.A_off && in_16bit(p) && bf16_mfma_eligible(p);
}

hipError_t launch_stream_form(const Problem &p, int tile)
{
    return p.in_f16 ? launch_tile<KIND_F16>(p, tile) : launch_tile<KIND_BF16>(p, tile);
}

}  // namespace brg
