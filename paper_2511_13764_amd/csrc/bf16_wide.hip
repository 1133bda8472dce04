// The 128 x 256 tile of the 128-row streaming kernel (bf16_stream128.hpp): four waves multiply,
// 64 x 128 each, four load; a three-stage ring of 48 KiB blocks.
//
// What it is for: 257 to 512 tiles of 128 x 128 need two workgroups of the two-stage kernel on
// most CUs, and 256 x 256 tiles leave half of the chip idle; as 128 x 256 they fit it in one round,
// with a quarter fewer bytes from L2 per flop than 128 x 128.
// What bounds it: the matrix pipe at the clock the chip holds.  2048 x 4096 x 4096 (NT) took 61 us in the run that took it apart,
// 50 without loads and fragment reads (54 without loads, 57 without reads); with 128 workgroups
// 49 and 40.  The LDS is next: 96 KiB of fragment reads and 48 KiB of writes per block, 1,150
// cycles of it against 1,024 of the matrix pipe.
// Measured, two-stage 128 x 128 -> this (us): NN 2304^3 36.1 -> 31.8, 2560^3 42.4 -> 35.8, 2816^3 50.2 ->
// 42.2; NT 1300 x 4096 x 4096 55.0 -> 48.9, 2048 x 4096 x 4096 68.4 -> 58.3, 576 x 11008 x 4096 62.2 -> 52.7;
// int8 2048 x 4096 x 4096 40.9 -> 34.6.
#include "bf16_stream128.hpp"

namespace brg {

namespace {

template <int KIND>
void (*pick_unpacked(const Problem &p))(Bf16Args)
{
    if (p.transA == 0)
        return p.transB == 1 ? bf16_stream128_kernel<true, LAY_K, KIND, 256> : bf16_stream128_kernel<true, LAY_MN, KIND, 256>;
    return p.transB == 1 ? bf16_stream128_kernel<false, LAY_K, KIND, 256> : bf16_stream128_kernel<false, LAY_MN, KIND, 256>;
}

template <int KIND>
void (*pick(const Problem &p))(Bf16Args)
{
    if (!p.b_packed)
        return pick_unpacked<KIND>(p);
    return p.transA == 0 ? bf16_stream128_kernel<true, LAY_PACKED, KIND, 256> : bf16_stream128_kernel<false, LAY_PACKED, KIND, 256>;
}

}  // namespace

// More 128 x 128 tiles than CUs, no more 128 x 256 ones (with fewer of the former the streaming kernels
// have a CU for each: 1024 x 4096 x 4096 34.4 against 47.7 us; with more of the latter 256 x 256 tiles win:
// 3072^3 55.6 against 80).  A few blocks are over before the deeper start is paid: 3072 x 2048 x 128 11.0
// against 11.7 us, K = 512 15.9 against 15.7.  FP8's 128-deep instruction takes a whole block at once.
bool wide_tile_wins(const Problem &p)
{
    const int64_t tm = (p.M + 127) / 128, tn = (p.N + 127) / 128;
    return (in_16bit(p) || p.in_s8) && tm * tn * p.nmat > 256 && tm * ((p.N + 255) / 256) * p.nmat <= 256 &&
           p.batch * (p.K / (p.in_s8 ? 128 : 64)) >= 8;
}

hipError_t launch_bf16_wide(const Problem &p)
{
    void (*kern)(Bf16Args) = p.in_s8 ? pick_unpacked<KIND_S8>(p) : p.in_f16 ? pick<KIND_F16>(p) : pick<KIND_BF16>(p);
    return stream128_launch<256>(kern, p);
}

}  // namespace brg
