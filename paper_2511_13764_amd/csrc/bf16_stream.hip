// bf16 GEMM kernels for few rows of A (skinny M: the M = 16 / 128 shapes of an MLP
// layer), where the time goes into streaming the B matrix from HBM once, not into the
// matrix pipe - the regime the paper describes as bound by memory bandwidth
// (Section 6, discussion of the flat-layout results) - and for grids of at most 256
// tiles of 128 x 128 (one workgroup per CU anyway: the 1024^3 and 2048^3 squares, the
// batch-reduce tiles).
//
// bf16_stream_kernel: a workgroup of 4 or 8 wavefronts owns a BM x 128 block of C
// (BM = 32 or 64; 128 only for FP8) and walks its share of K in 64-deep blocks.  What
// matters here is how many bytes are in flight per CU, so the LDS is a ring of three
// stages, each holding one k-block of A and B: the loads for block t + 2 are requested
// while block t is multiplied, and the small footprint (60 to 96 KiB) lets a second
// workgroup share the CU.  (Sweeps of 2 to 8 stages on the MLP shapes: three is best
// or within 3 % of the best everywhere; deeper rings lose the second workgroup and
// gain nothing.)  Loads are global->LDS DMA (no register staging), counted per wave
// with vmcnt: before block t is read a wave waits until only the loads of block t + 1
// are outstanding, then one workgroup barrier publishes the block and frees the slot
// read in the previous iteration.
//
// bf16_stream128_kernel: the 128-row tile, with loading and multiplying given to
// different waves (described at the kernel).
#include "bf16_stream128.hpp"

namespace brg {

namespace {

constexpr int ST_BN = 128;
constexpr int ST_STAGES = 3;

// Waves per workgroup: 8 (two per SIMD) for the 128- and 64-row tiles - twice as many
// waves issuing the global->LDS loads raises what one CU can pull (measured 77-96
// against 57 B/ns) and these shapes are bound by exactly that; 4 for the 32-row tile,
// whose A block is only 4 wave-loads.
template <int BM>
struct StreamWaves { static constexpr int value = BM >= 64 ? 8 : 4; };

// STAGES: depth of the LDS ring (three, see above; a six-deep ring for batch-reduce
// calls over scattered tiles measured the same as three: there the time is a chain of
// fixed latencies - launch, offsets, first tiles, partial tiles, second launch).
template <int BM, bool A_KMAJ, int B_LAY, int KIND, int STAGES = ST_STAGES>
__global__ void __launch_bounds__(StreamWaves<BM>::value * 64)
bf16_stream_kernel(Bf16Args p)
{
    constexpr int NW = StreamWaves<BM>::value;
    static_assert(A_KMAJ || BM == 128, "an m-contiguous A needs the 128-row tile");
    typedef typename TileOf<BM, NW, A_KMAJ ? LAY_K : LAY_MN, KIND>::type ATile;
    typedef typename TileOf<ST_BN, NW, B_LAY, KIND>::type BTile;
    constexpr int WGM = BM == 128 ? 2 : 1, WGN = NW / WGM;    // wave grid
    constexpr int WM = BM / WGM, WN = ST_BN / WGN;
    constexpr int TM = WM / 16, TN = WN / 16;                 // 16x16 MFMA tiles per wave
    constexpr uint32_t A_BYTES = BM * BK * 2, B_BYTES = ST_BN * BK * 2;
    constexpr uint32_t STAGE = A_BYTES + B_BYTES;
    constexpr int L = ATile::kPerWave + BTile::kPerWave;        // loads per wave per block
    constexpr int stages = STAGES;
    static_assert((STAGES - 2) * L <= 63, "outstanding loads must fit vmcnt");

    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    LDS_AS char *smem = (LDS_AS char *)smem_generic;
    select_matrix(p);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WGN, wn = w % WGN;

    int tile, slice;
    slice_major_coords(p.tiles_m * p.tiles_n, p.split, p.walk, tile, slice);
    const int tn = div_by(tile, p.walk.by_group), tm = tile - tn * p.tiles_m;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * ST_BN;

    // Reduction range of this workgroup: flattened (batch, k-block) iterations.
    const int kblocks = (int)(p.K / BK);
    const int total = (int)p.batch * kblocks;
    const int per = (int)p.walk.per;
    const int it_begin = slice * per;
    const int it_end = (it_begin + per < total) ? it_begin + per : total;
    const int n_iter = it_end > it_begin ? it_end - it_begin : 0;

    // Rows / columns past the edge of the matrix are redirected to a valid one (their
    // products land in accumulator rows / columns that are never stored), so every
    // wave issues exactly L loads per block and the vmcnt arithmetic below holds.
    uint32_t a_src[ATile::kPerWave], b_src[BTile::kPerWave];
#pragma unroll
    for (int j = 0; j < ATile::kPerWave; ++j)
        a_src[j] = ATile::src_rel_bytes(w, j, lane, m0, p.M, p.lda);
#pragma unroll
    for (int j = 0; j < BTile::kPerWave; ++j)
        b_src[j] = BTile::src_rel_bytes(w, j, lane, n0, p.N, p.ldb);
    const int64_t b_kstep = BTile::kstep(p.ldb);
    const int64_t a_kstep = ATile::kstep(p.lda);
    const int64_t a_origin = ATile::origin(m0, p.lda), b_origin = BTile::origin(n0, p.ldb);
    // Load cursor: (batch index, k-block) of the next block to request and its pointers.
    int ld_i = n_iter > 0 ? div_by(it_begin, p.walk.by_kblocks) : 0;
    int ld_kb = n_iter > 0 ? it_begin - ld_i * kblocks : 0;
    // (where it starts its turn of the blocks, and where that wraps)
    const bool rotate = A_KMAJ && B_LAY == LAY_K && p.rotate && n_iter > 1;
    const int wrap = rotate ? it_end : kblocks;
    if (rotate) {
        const int at = tn - div_by(tn, p.walk.by_per) * (int)p.walk.per;
        ld_kb += at < n_iter ? at : 0;
    }
    TileOffsets offs_a, offs_b;                 // this wave's window of the tile offsets
    // Tile offsets live in device memory: if one of this workgroup's tiles does not
    // start at a multiple of 8 elements the workgroup stages its blocks through
    // registers with 2-byte loads instead (same LDS image; those loads complete before
    // the stores, so the counted waits below simply find nothing outstanding).  Every
    // wave looks at all of the workgroup's tiles (the first 64 are the window it keeps),
    // so all waves reach the same verdict without a barrier.
    bool direct = true;
    if (p.A_off) {
        offs_a.init(p.A_off, p.batch, ld_i, lane);
        offs_b.init(p.B_off, p.batch, ld_i, lane);
        const int last_i = n_iter > 0 ? div_by(it_end - 1, p.walk.by_kblocks) : ld_i;
        int bad = (ld_i + lane <= last_i) && (((offs_a.lo | offs_b.lo) & 7u) != 0);
        for (int i = ld_i + 64 + lane; i <= last_i; i += 64)
            bad |= (((p.A_off[i] | p.B_off[i]) & 7) != 0);
        direct = __builtin_amdgcn_ballot_w64(bad != 0) == 0;
    }
    const uint16_t *ld_a = uniform_ptr(p.A + (p.A_off ? offs_a.get(ld_i, lane) : 0) + a_origin + ld_kb * a_kstep);
    const uint16_t *ld_b = uniform_ptr(p.B + (p.B_off ? offs_b.get(ld_i, lane) : 0) + b_origin + ld_kb * b_kstep);
    int ld_slot = 0;
    auto staged16 = [&](const char *gc, uint32_t lds_byte) {
        const uint16_t *g = (const uint16_t *)gc;
        s16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = (short)g[e];
        *(LDS_AS s16x8 *)(smem + lds_byte + lane * 16) = v;
    };

    auto issue_loads = [&]() {
        const uint32_t base = (uint32_t)ld_slot * STAGE;
        if (direct) {
#pragma unroll
            for (int j = 0; j < BTile::kPerWave; ++j)
                load16_to_lds_saddr((const char *)ld_b, b_src[j],
                                    (uint32_t)(size_t)(smem + base + A_BYTES + BTile::dst_byte(w, j)));
#pragma unroll
            for (int j = 0; j < ATile::kPerWave; ++j)
                load16_to_lds_saddr((const char *)ld_a, a_src[j],
                                    (uint32_t)(size_t)(smem + base + ATile::dst_byte(w, j)));
        } else {
#pragma unroll
            for (int j = 0; j < BTile::kPerWave; ++j)
                staged16((const char *)ld_b + b_src[j], base + A_BYTES + BTile::dst_byte(w, j));
#pragma unroll
            for (int j = 0; j < ATile::kPerWave; ++j)
                staged16((const char *)ld_a + a_src[j], base + ATile::dst_byte(w, j));
        }
        if (++ld_kb == wrap) {
            ld_kb = rotate ? it_begin : 0;
            ++ld_i;
            if (rotate) {
                ld_a -= (n_iter - 1) * a_kstep;
                ld_b -= (n_iter - 1) * b_kstep;
            }
            if (p.A_off && ld_i < (int)p.batch) {
                ld_a = uniform_ptr(p.A + offs_a.get(ld_i, lane) + a_origin);
                ld_b = uniform_ptr(p.B + offs_b.get(ld_i, lane) + b_origin);
            }
        } else {
            ld_a += a_kstep;
            ld_b += b_kstep;
        }
        ld_slot = ld_slot + 1 == stages ? 0 : ld_slot + 1;
    };
    f32x4 acc[TN][TM];
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
            acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    const int ahead = stages - 1;
    for (int s = 0; s < ahead && s < n_iter; ++s)
        issue_loads();

    // The MFMAs of the second 32-deep half of a block are issued at the top of the next
    // iteration, so the matrix pipe works through the wait for the next block, the barrier
    // and the load requests.  (Not for FP8: its 128-deep instruction needs both halves.)
    bf16x8 fa[2][TM], fb[2][TN];
    auto mfma_half = [&](auto hc) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[a][b] = mfma_16x16x32<kind_is_f8(KIND) ? KIND_BF16 : KIND>(fb[h][a], fa[h][b], acc[a][b]);
    };
    constexpr std::integral_constant<int, 0> H0{};
    constexpr std::integral_constant<int, 1> H1{};
    int rd_slot = 0;
    for (int t = 0; t < n_iter; ++t) {
        if constexpr (!kind_is_f8(KIND)) {
            if (t > 0)
                mfma_half(H1);                      // second half of block t - 1
            __builtin_amdgcn_sched_barrier(0);
        }
        // Block t has landed once only the stages - 2 younger blocks are outstanding.
        if (t + stages - 2 < n_iter)
            wait_vmcnt_le<(STAGES - 2) * L>();
        else
            wait_vmcnt0();                          // tail: fewer blocks than slots remain
        if (!direct)
            wait_lgkmcnt0();                        // register-staged blocks: their LDS stores
        block_sync();
        if (t + ahead < n_iter)
            issue_loads();                          // into the slot read in iteration t - 1
        LDS_AS char *at = smem + (uint32_t)rd_slot * STAGE;
        LDS_AS char *bt = at + A_BYTES;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
#pragma unroll
            for (int i = 0; i < TM; ++i)            // FP8: st = which half of a lane's 32-byte operand
                fa[st][i] = ATile::read_frag16(at, wm * WM, i, st, lane);
#pragma unroll
            for (int i = 0; i < TN; ++i)
                fb[st][i] = BTile::read_frag16(bt, wn * WN, i, st, lane);
        }
        if constexpr (kind_is_f8(KIND)) {
#pragma unroll
            for (int a = 0; a < TN; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[a][b] = mfma_16x16x128_f8<KIND>(fb[0][a], fb[1][a], fa[0][b], fa[1][b], acc[a][b]);
        } else {
            mfma_half(H0);
        }
        // The fragments are in registers before the next barrier lets another wave's
        // loads overwrite this slot.
        wait_lgkmcnt0();
        rd_slot = rd_slot + 1 == stages ? 0 : rd_slot + 1;
    }
    if constexpr (!kind_is_f8(KIND)) {
        if (n_iter > 0)
            mfma_half(H1);
    }

    store_wave_tile16<TM, TN>(p, acc, m0 + wm * WM + (lane & 15), n0 + wn * WN + 4 * (lane >> 4), slice);
}

template <int BM>
hipError_t launch_stream(const Problem &p)
{
    Bf16Args a;
    fill_common_args(a, p);
    a.tiles_m = (int)((p.M + BM - 1) / BM);
    a.tiles_n = (int)((p.N + ST_BN - 1) / ST_BN);
    const bool by_kind = BM == 128 && !p.in_f8;     // bf16_stream128_kernel, which walks groups
    a.walk = make_walk(a.tiles_m, a.tiles_n, p.split, a.K / BK, p.batch, by_kind ? (int64_t)kWalkRows * a.tiles_n : a.tiles_m);
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)p.split, (unsigned)p.nmat);
    void (*kern)(Bf16Args) = nullptr;
    size_t lds = (size_t)ST_STAGES * (BM + ST_BN) * BK * 2;
    // One-byte operands come unpacked in all four layouts; 16-bit ones also with a packed B.
#define BRG_ST_B(AK, KIND)                                                                    \
    kern = p.transB == 1 ? bf16_stream_kernel<BM, AK, LAY_K, KIND> : bf16_stream_kernel<BM, AK, LAY_MN, KIND>;
#define BRG_ST_B3(AK, KIND)                                                                   \
    kern = p.b_packed ? bf16_stream_kernel<BM, AK, LAY_PACKED, KIND>                           \
           : p.transB == 1 ? bf16_stream_kernel<BM, AK, LAY_K, KIND> : bf16_stream_kernel<BM, AK, LAY_MN, KIND>;
#define BRG_S128_B(AK, KIND)                                                                  \
    kern = p.transB == 1 ? bf16_stream128_kernel<AK, LAY_K, KIND> : bf16_stream128_kernel<AK, LAY_MN, KIND>;
#define BRG_S128_B3(AK, KIND)                                                                 \
    kern = p.b_packed ? bf16_stream128_kernel<AK, LAY_PACKED, KIND>                            \
           : p.transB == 1 ? bf16_stream128_kernel<AK, LAY_K, KIND> : bf16_stream128_kernel<AK, LAY_MN, KIND>;
    if constexpr (BM == 128) {
        // Everything but FP8 takes the loader / multiplier form of the 128-row tile.
        if (p.in_f8) {
            if (p.transA == 0) {
                if (p.f8_e5m2) { BRG_ST_B(true, KIND_BF8) } else { BRG_ST_B(true, KIND_F8) }
            } else {
                if (p.f8_e5m2) { BRG_ST_B(false, KIND_BF8) } else { BRG_ST_B(false, KIND_F8) }
            }
        } else {
            lds = S128<128>::kLds;
            if (p.transA == 0) {
                if (p.in_s8) { BRG_S128_B(true, KIND_S8) }
                else if (p.in_f16) { BRG_S128_B3(true, KIND_F16) } else { BRG_S128_B3(true, KIND_BF16) }
            } else {
                if (p.in_s8) { BRG_S128_B(false, KIND_S8) }
                else if (p.in_f16) { BRG_S128_B3(false, KIND_F16) } else { BRG_S128_B3(false, KIND_BF16) }
            }
        }
    } else {
        if (p.transA != 0)
            return hipErrorInvalidValue;            // the 32- and 64-row tiles need a k-contiguous A
        if (p.in_s8) {
            BRG_ST_B(true, KIND_S8)
        } else if (p.in_f8) {
            if (p.f8_e5m2) { BRG_ST_B(true, KIND_BF8) } else { BRG_ST_B(true, KIND_F8) }
        } else if (p.in_f16) {
            BRG_ST_B3(true, KIND_F16)
        } else {
            BRG_ST_B3(true, KIND_BF16)
        }
    }
#undef BRG_ST_B
#undef BRG_ST_B3
#undef BRG_S128_B
#undef BRG_S128_B3
    static thread_local const void *configured[40] = {nullptr};
    bool done = false;
    for (const void *c : configured)
        done = done || c == (const void *)kern;
    if (!done) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
        for (auto &c : configured)
            if (!c) { c = (const void *)kern; break; }
    }
    hipLaunchKernelGGL(kern, grid, dim3(StreamWaves<BM>::value * 64), lds, p.stream, a);
    return hipGetLastError();
}

}  // namespace

// The 48-column form of the 128-row kernel.
hipError_t launch_bf16_stream_narrow(const Problem &p)
{
    return stream128_launch<48>(p.in_f16 ? bf16_stream128_kernel<true, LAY_K, KIND_F16, 48> : bf16_stream128_kernel<true, LAY_K, KIND_BF16, 48>, p);
}

// The tile of as many elements that the automatic plan takes for a plain 16-bit product instead of the 32- and 64-row variants' own, or -1.  64 x 64 pulls 16 KiB per
// block where 32 x 128 pulls 20, and its loading waves never wait for its multiplying ones, but a short reduction ends before its deeper start
// is paid back: of 700 problems with up to 256 of its tiles 1.01 to 1.02 of the time with K up to 384, 0.99 to 512, 0.95 to 640, 0.91 to 1024, 0.84 to 2048,
// 0.78 beyond; with more tiles 0.90 to 1.00 from 512 on, 1.08 below.  128 x 64 against 64 x 128, which pull the same: with up to 256 tiles 1.16 with K
// up to 320, 1.04 to 1024, 0.96 to 1536, 0.91 to 2048, 0.85 beyond; with more 1.02 to 1.24 everywhere.
int stream_tile_instead(const Problem &p, int bm, int split)
{
    if (!in_16bit(p) || p.batch != 1 || p.A_off || p.transA || split != 1 || p.M <= bm)
        return -1;
    if (bm == 32)
        return p.K >= 512 ? GEN_64 : -1;
    return bm == 64 && p.K >= 1280 && ((p.M + 127) / 128) * ((p.N + 63) / 64) * p.nmat <= 256 ? GEN_MID : -1;
}

hipError_t launch_bf16_stream(const Problem &p, int bm)
{
    switch (bm) {
    case 32: return launch_stream<32>(p);
    case 64: return launch_stream<64>(p);
    case 128: return launch_stream<128>(p);
    default: return hipErrorInvalidValue;
    }
}

// The 32- and 64-row tiles need A stored M x K (k contiguous), the 128-row tile takes
// either order; B in any layout; batch-reduce with tile offsets included.
bool bf16_stream_eligible(const Problem &p, int bm)
{
    return bf16_mfma_eligible(p) && (p.transA == 0 || bm == 128);
}

}  // namespace brg
