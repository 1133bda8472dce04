// The 128-row streaming kernel: four waves load, four multiply.  Tiles of 128 x 128 and 128 x 48
// (bf16_stream.hip) and 128 x 256 (bf16_wide.hip).
#pragma once
#include "bf16_tiles.hpp"

namespace brg {

namespace {

// ---------------------------------------------------------------------------
// 128 x 128 tile with the work divided by kind: four waves multiply, four waves load.
//
// What bounds a 128 x 128 x 64 block on one CU (cycles per block, measured with
// work-skipping copies of bf16_stream_kernel (bf16_stream.hip) and with s_memtime around its steps):
// the matrix pipe needs 512 per SIMD; eight waves reading the fragments of 64 x 32
// accumulator tiles need 600-1100 (96 KiB of LDS reads, a SIMD takes its share at
// about 32 B/clk); the 32 global->LDS wave-loads need about 780 (a CU pulls at
// most ~42 B/clk from L2 with every CU pulling), and a wave is held at each of its
// loads until the address unit has taken it.  In that kernel all of that is
// serial: every wave requests loads, reads fragments, then multiplies - 0.63 us per
// block where the loads alone need 0.34.
//
// Here waves 0-3 (one per SIMD) own 64 x 64 accumulator tiles (64 KiB of fragment
// reads per block) and never touch global memory inside the loop; waves 4-7 (the
// second wave of every SIMD) only request loads, eight per block each, and wait
// for them.  One workgroup barrier per block, B(t), publishes block t and frees
// the slot of block t - 1, into which the loaders then request block t + STAGES - 1.
// A multiplying wave reads the fragments of the first 32-deep half of block t
// while the matrix pipe works on the second half of block t - 1, and those of the
// second half while it works on the first, so the pipe only idles for the barrier.
//
// BN = 48: a weight stream (81 to 128 rows of A, N around 11008) whose 128-column tiles
// leave CUs without work unless the reduction is split.  A workgroup pulls 16 KiB of A and
// 6 KiB of B per block (70 B/ns), six stages keep 30 KiB of B requested per CU, and no
// partial tiles are written: 128 x 11008 x 4096 31.4 -> 28.3 us, 128 x 9216 x 2048 16.3 -> 13.8.
// The B image keeps 64 rows (whole wave-loads per loader); the last 16 repeat row 47.
// ---------------------------------------------------------------------------
#ifndef BRG_ST128_STAGES
#define BRG_ST128_STAGES 4
#endif
constexpr int S128_STAGES = BRG_ST128_STAGES;

// Columns of the tile: 128; 48 for a weight stream that 128-column tiles leave on too few
// CUs; 256 where two rounds' worth of 128-column tiles fit the chip at once as half as many.  Pitch of a staged row: 4 floats more (528 B: conflict-free 16-byte writes).
template <int BN, int BM = 128> struct S128 {
    static constexpr int kLoadRows = BN >= 64 ? BN : 64;          // B rows per stage, whole wave-loads per loader
    static constexpr int kStages = BN == 256 || (BN == 64 && BM == 128) ? 3 : BN == 48 ? 6 : S128_STAGES;
    static constexpr uint32_t kStage = (BM + kLoadRows) * BK * 2;
    static constexpr size_t kLds = (size_t)kStages * kStage;
};

// All 512 threads: the staged fp32 tile, whole rows per wave and instruction, to C (beta,
// bias, ReLU, narrowing) or to this split's partial sums.  The old values of an accumulating
// fp32 C, and its bias, are requested when the kernel starts (2048 x 2048 x 256 with beta = 1: 10.4 ->
// 9.5 us; with bias and ReLU 11.2 -> 9.5, and 12.8 when only the old values were).  They come
// before the loaders' first block and so hold it up, but no second workgroup follows on a CU.
template <int BN, int BM = 128>
struct S128Store {
    static constexpr int LD = BN + 4, QUADS = BN / 4, N_IT = BM * QUADS / 512;
    static constexpr int N_BIAS = 512 % QUADS == 0 ? 1 : N_IT;    // a thread's columns: the same for all its rows, or not
    static constexpr int kPieces = BN == 64 ? PIECES_32BIT : PIECES_NONE;
    static constexpr bool kEarly = BN < 256;    // (at 256 columns the accumulators leave no registers for them before the loop ends)
    f32x4 old[N_IT], bias[N_BIAS];
    bool accumulate;

    __device__ __forceinline__ void begin(const Bf16Args &p, int tid, int64_t m0, int64_t n0)
    {
        accumulate = accumulates_f32(p.epi, p.split > 1) && n0 + BN <= p.N;
        if (kEarly && accumulate)
            request(p, tid, m0, n0);
    }
    __device__ __forceinline__ void request(const Bf16Args &p, int tid, int64_t m0, int64_t n0)
    {
#pragma unroll
        for (int i = 0; i < N_IT; ++i) {
            const int idx = i * 512 + tid;
            const int64_t m = m0 + idx / QUADS;
            old[i] = *(const f32x4 *)((const float *)p.epi.C + (m < p.M ? m : p.M - 1) * p.epi.ldc + n0 + (idx % QUADS) * 4);
            if (i < N_BIAS)
                bias[i] = bias4(p.epi, n0 + (idx % QUADS) * 4);
        }
    }
    __device__ __forceinline__ void store(const Bf16Args &p, LDS_AS char *smem, int tid, int64_t m0, int64_t n0, int slice)
    {
        LDS_AS float *stage = (LDS_AS float *)smem;
        if (accumulate) {
            if (!kEarly)
                request(p, tid, m0, n0);
#pragma unroll
            for (int i = 0; i < N_IT; ++i) {
                const int idx = i * 512 + tid;
                const int row = idx / QUADS, c4 = idx % QUADS;
                if (m0 + row < p.M)
                    store4_accumulated(p.epi, m0 + row, n0 + c4 * 4, old[i], bias[i % N_BIAS],
                                       *(LDS_AS f32x4 *)(stage + row * LD + c4 * 4));
            }
            return;
        }
        const bool to_partial = p.split > 1;
        float *part = to_partial ? p.partial + (int64_t)slice * p.M * p.N : nullptr;
        const bool vec = to_partial ? ((p.N & 3) == 0) : ((p.epi.ldc & 3) == 0 && (((uintptr_t)p.epi.C) & 15) == 0);
#pragma unroll 2
        for (int i = 0; i < N_IT; ++i) {
            const int idx = i * 512 + tid;
            const int row = idx / QUADS, c4 = idx % QUADS;
            const f32x4 v = *(LDS_AS f32x4 *)(stage + row * LD + c4 * 4);
            const int64_t m = m0 + row, n = n0 + c4 * 4;
            if (m < p.M && n < p.N) {
                if (to_partial)
                    store4_partial<kPieces>(part + m * p.N + n, p.N - n, vec, v[0], v[1], v[2], v[3]);
                else
                    store4_epilogue<kPieces>(p.epi, m, n, p.N - n, vec, v[0], v[1], v[2], v[3]);
            }
        }
    }
};

// TAIL: K is no multiple of 64 (16-bit operands).  A block of kt < 64 k-values that ends the reduction is taken FIRST
// (unsplit, or by the first slice): block 0 stands for it, block t for the whole block t - 1.  Instances of
// their own: as a branch of the plain ones it cost those 4 to 6 scalar spills.  These calls are the general path's, whose
// sums are not one chain of fp32 additions over all of K, and so what the accumulators hold is added to totals every
// 16 blocks, where the sum stays in fp32 and the tile leaves registers for it (not at 256 columns): 2 % of such a call, and 0.64 to
// 0.78 of the error of one chain.
// BN = 64: 64 x 64 and 128 x 64 tiles (bf16_stream64.hip), small enough for two workgroups on a CU.
// TOTAL: sums that are not one chain, as above; the 64-column tiles have two, and close off every fourth block.
template <bool A_KMAJ, int B_LAY, int KIND, int BN = 128, bool TAIL = false, int BM = 128, bool TOTAL = TAIL && BN < 256>
__global__ void __launch_bounds__(512, BN == 64 && !(BM == 128 && TOTAL) ? 4 : 2)
bf16_stream128_kernel(Bf16Args p)
{
    static_assert(!TAIL || !kind_is_8bit(KIND), "");
    constexpr int NL = 4;                        // loader waves
    static_assert(!kind_is_f8(KIND), "the 128-deep FP8 instruction takes a whole k-block");
    typedef typename TileOf<BM, NL, A_KMAJ ? LAY_K : LAY_MN, KIND>::type ATile;
    static_assert(BN != 48 || (A_KMAJ && B_LAY == LAY_K && BM == 128), "the narrow tile is for k-contiguous operands");
    typedef S128<BN, BM> Cfg;
    typedef typename TileOf<Cfg::kLoadRows, NL, B_LAY, KIND>::type BTile;
    constexpr int WM = BN == 48 ? 32 : BM / 2, WN = BN == 48 ? BN : BN / 2, TM = WM / 16, TN = WN / 16;
    constexpr uint32_t A_BYTES = BM * BK * 2, STAGE = Cfg::kStage;
    constexpr int LA = ATile::kPerWave, LB = BTile::kPerWave, L = LA + LB;
    constexpr int stages = Cfg::kStages, ahead = stages - 1;
    static_assert(L == (BM + Cfg::kLoadRows) / 32 && (stages - 2) * L <= 63, "outstanding loads must fit vmcnt");

    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    LDS_AS char *smem = (LDS_AS char *)smem_generic;
    select_matrix(p);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    int tile, slice, tm, tn;
    slice_major_coords(p.tiles_m * p.tiles_n, p.split, p.walk, tile, slice);
    group_walk(tile, p.tiles_m, p.tiles_n, p.walk, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    const int kt = TAIL ? (int)(p.K % BK) : 0;
    const int kblocks = (int)(p.K / BK) + (TAIL ? 1 : 0);
    const int total = (int)p.batch * kblocks;
    const int per = (int)p.walk.per;
    const int it_begin = slice * per;
    const int it_end = (it_begin + per < total) ? it_begin + per : total;
    const int n_iter = it_end > it_begin ? it_end - it_begin : 0;

    // A tile offset that is not a multiple of 8 elements sends the loaders to
    // register-staged 2-byte loads (same LDS image; they complete before their LDS
    // stores, so the counted waits find nothing outstanding).
    bool direct = true;
    if (p.A_off) {
        int ok = 1;
        for (int i = tid; i < (int)p.batch; i += 512)
            ok &= (((p.A_off[i] | p.B_off[i]) & 7) == 0);
        direct = __syncthreads_and(ok) != 0;
    }

    S128Store<BN, BM> out;
    out.begin(p, tid, m0, n0);

    if (w >= 4) {
        // ---------------- loader waves ----------------
        const int wl = w - 4;
        // Rows / columns past the edge are redirected to a valid one (their products
        // land in accumulator rows / columns that are never stored), so every wave
        // issues exactly L loads per block and the vmcnt arithmetic holds.
        uint32_t a_src[LA], b_src[LB];
#pragma unroll
        for (int j = 0; j < LA; ++j)
            a_src[j] = ATile::src_rel_bytes(wl, j, lane, m0, p.M, p.lda);
#pragma unroll
        for (int j = 0; j < LB; ++j)
            b_src[j] = BTile::src_rel_bytes(wl, j, lane, n0, BN != 48 || p.N < n0 + BN ? p.N : n0 + BN, p.ldb);
        const int64_t b_kstep = BTile::kstep(p.ldb);
        const int64_t a_kstep = ATile::kstep(p.lda);
        const int64_t a_origin = ATile::origin(m0, p.lda), b_origin = BTile::origin(n0, p.ldb);
        int ld_i = n_iter > 0 ? div_by(it_begin, p.walk.by_kblocks) : 0;
        int ld_kb = n_iter > 0 ? it_begin - ld_i * kblocks : 0;
        // (where it starts its turn of the blocks, and where that wraps)
        const bool rotate = !TAIL && A_KMAJ && B_LAY == LAY_K && p.rotate && n_iter > 1;
        const int wrap = rotate ? it_end : kblocks;
        if (rotate) {
            const int at = tn - div_by(tn, p.walk.by_per) * (int)p.walk.per;
            ld_kb += at < n_iter ? at : 0;
        }
        const int ld_first = TAIL && ld_kb > 0 ? ld_kb - 1 : ld_kb;
        TileOffsets offs_a, offs_b;             // this wave's window of the tile offsets
        if (p.A_off) {
            offs_a.init(p.A_off, p.batch, ld_i, lane);
            offs_b.init(p.B_off, p.batch, ld_i, lane);
        }
        const uint16_t *ld_a = uniform_ptr(p.A + (p.A_off ? offs_a.get(ld_i, lane) : 0) + a_origin + ld_first * a_kstep);
        const uint16_t *ld_b = uniform_ptr(p.B + (p.B_off ? offs_b.get(ld_i, lane) : 0) + b_origin + ld_first * b_kstep);
        int ld_slot = 0;
        auto issue_one = [&](const char *base, uint32_t src, uint32_t dst) {
            if (direct) {
                load16_to_lds_saddr(base, src, (uint32_t)(size_t)(smem + dst));
            } else {
                const uint16_t *h = (const uint16_t *)(base + src);
                s16x8 v;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = (short)h[e];
                *(LDS_AS s16x8 *)(smem + dst + lane * 16) = v;
            }
        };
        auto issue_block = [&]() {
            const uint32_t base = (uint32_t)ld_slot * STAGE;
#pragma unroll
            for (int j = 0; j < LB; ++j)
                issue_one((const char *)ld_b, b_src[j], base + A_BYTES + BTile::dst_byte(wl, j));
#pragma unroll
            for (int j = 0; j < LA; ++j)
                issue_one((const char *)ld_a, a_src[j], base + ATile::dst_byte(wl, j));
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
        int requested = 0;
        if constexpr (TAIL) {
            if (it_begin == 0 && n_iter > 0) {
                // The incomplete block, through registers, behind the requests of those that follow it.
                ld_slot = 1;
                ++ld_kb;
                for (requested = 1; requested < ahead && requested < n_iter; ++requested)
                    issue_block();
                const char *ta = (const char *)(p.A + a_origin + (kblocks - 1) * a_kstep);
                const char *tb = (const char *)(p.B + b_origin + (kblocks - 1) * b_kstep);
                s16x8 v[L];
#pragma unroll
                for (int j = 0; j < LA; ++j)
                    v[j] = ATile::tail_chunk(ta + a_src[j], wl * LA + j, lane, kt, p.lda);
#pragma unroll
                for (int j = 0; j < LB; ++j)
                    v[LA + j] = BTile::tail_chunk(tb + b_src[j], wl * LB + j, lane, kt, p.ldb);
#pragma unroll
                for (int j = 0; j < LA; ++j)
                    *(LDS_AS s16x8 *)(smem + ATile::dst_byte(wl, j) + lane * 16) = v[j];
#pragma unroll
                for (int j = 0; j < LB; ++j)
                    *(LDS_AS s16x8 *)(smem + A_BYTES + BTile::dst_byte(wl, j) + lane * 16) = v[LA + j];
            }
        }
        for (; requested < ahead && requested < n_iter; ++requested)
            issue_block();
        for (int t = 0; t < n_iter; ++t) {
            // Block t has landed once only the stages - 2 younger blocks are outstanding.
            if (t + ahead - 1 < n_iter)
                wait_vmcnt_le<(stages - 2) * L>();
            else
                wait_vmcnt0();                      // tail: fewer blocks than slots remain
            wait_lgkmcnt0();                        // register-staged blocks: their LDS stores
            block_sync();                           // B(t)
            if (t + ahead < n_iter)
                issue_block();                      // into the slot of block t - 1
        }
        block_sync();                               // E1
        block_sync();                               // E2: the staged tile is complete
        out.store(p, smem, tid, m0, n0, slice);
        return;
    }

    // ---------------- multiplying waves ----------------
    const int wm = BN == 48 ? w : w >> 1, wn = BN == 48 ? 0 : w & 1;
    constexpr bool TOTALS = TOTAL;
    constexpr int CHAINS = TOTAL && BN == 64 ? 2 : 1;       // one for each half of a block
    constexpr int EVERY = BN == 64 ? 4 : 16;        // blocks between additions to the totals
    f32x4 acc[CHAINS][TN][TM];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[c][a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto chains = [&](int a, int b) {
        if constexpr (CHAINS == 2)
            return acc[0][a][b] + acc[1][a][b];
        else
            return acc[0][a][b];
    };
    const bool with_totals = TOTALS && (p.split > 1 || p.epi.c_f32);
    f32x4 closed[TOTALS ? TN : 1][TOTALS ? TM : 1];
    bool any = false;                               // ... are there totals
    bf16x8 fa[2][TM], fb[2][TN];
    auto read_half = [&](LDS_AS char *at, LDS_AS char *bt, auto hc) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[h][i] = ATile::read_frag16(at, wm * WM, i, h, lane);
#pragma unroll
        for (int i = 0; i < TN; ++i)
            fb[h][i] = BTile::read_frag16(bt, wn * WN, i, h, lane);
    };
    auto mfma_half = [&](auto hc) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[h % CHAINS][a][b] = mfma_16x16x32<KIND>(fb[h][a], fa[h][b], acc[h % CHAINS][a][b]);
    };
    constexpr std::integral_constant<int, 0> H0{};
    constexpr std::integral_constant<int, 1> H1{};
    int rd_slot = 0;
    auto block = [&](auto first) {
        block_sync();                               // B(t): block t is in LDS
        LDS_AS char *at = smem + (uint32_t)rd_slot * STAGE;
        LDS_AS char *bt = at + A_BYTES;
        read_half(at, bt, H0);
        if constexpr (!decltype(first)::value)
            mfma_half(H1);                          // second half of block t - 1
        __builtin_amdgcn_sched_barrier(0);
        read_half(at, bt, H1);
        mfma_half(H0);
        __builtin_amdgcn_sched_barrier(0);
        // Every read of block t is complete before the barrier that lets the loaders
        // overwrite its slot.
        wait_lgkmcnt0();
        rd_slot = rd_slot + 1 == stages ? 0 : rd_slot + 1;
    };
    if (n_iter > 0)
        block(std::true_type{});
    for (int t = 1; t < n_iter;) {
        // (a loop within a loop: a branch in every block took 3 % of the call)
        const int stop = with_totals && t + EVERY < n_iter ? t + EVERY : n_iter;
        for (; t < stop; ++t)
            block(std::false_type{});
        if constexpr (TOTALS) {
            if (t < n_iter) {
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b) {
                        closed[a][b] = any ? closed[a][b] + chains(a, b) : chains(a, b);
#pragma unroll
                        for (int c = 0; c < CHAINS; ++c)
                            acc[c][a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                any = true;
            }
        }
    }
    if (n_iter > 0)
        mfma_half(H1);
    if constexpr (CHAINS == 2) {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[0][a][b] = chains(a, b);
    }
    if (TOTALS && any) {
        asm volatile("");                           // (a branch)
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[0][a][b] += closed[TOTALS ? a : 0][TOTALS ? b : 0];
    }
    // Epilogue through LDS: written from the MFMA layout (lane l: row l % 16, columns
    // 4 * (l / 16) .. + 3 of each 16 x 16 tile), read back row-wise by all eight waves,
    // so that every store instruction covers whole rows of the tile instead of sixteen
    // 32-byte pieces (measured: 4 us of an 8 MiB C went into such stores).
    block_sync();                                   // E1: nobody reads fragments any more
    LDS_AS float *stage = (LDS_AS float *)smem;
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
            *(LDS_AS f32x4 *)(stage + (wm * WM + 16 * b + (lane & 15)) * (BN + 4) + wn * WN + 16 * a + 4 * (lane >> 4)) =
                acc[0][a][b];
    wait_lgkmcnt0();
    block_sync();                                   // E2
    out.store(p, smem, tid, m0, n0, slice);
}

// Launch one instance.
template <int BN, int BM = 128>
hipError_t stream128_launch(void (*kern)(Bf16Args), const Problem &p)
{
    Bf16Args a;
    fill_common_args(a, p);
    a.tiles_m = (int)((p.M + BM - 1) / BM);
    a.tiles_n = (int)((p.N + BN - 1) / BN);
    a.walk = make_walk(a.tiles_m, a.tiles_n, p.split, (a.K + BK - 1) / BK, p.batch, (int64_t)kWalkRows * a.tiles_n);
    if (BN == 48)                                   // (128 x 11008 x 4096, three matrices in turn: 27.0 us, rotated 27.2 to 28.3)
        a.rotate = 0;
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)p.split, (unsigned)p.nmat);
    constexpr size_t lds = S128<BN, BM>::kLds;
    static thread_local const void *configured[32] = {nullptr};
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
    hipLaunchKernelGGL(kern, grid, dim3(512), lds, p.stream, a);
    return hipGetLastError();
}

}  // namespace

}  // namespace brg
