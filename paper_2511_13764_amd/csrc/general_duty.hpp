// The general kernel's wide tiles with the work divided by kind: four or eight waves load, four
// multiply.  Included by general.hpp, whose loaders, LDS images and epilogue it uses.
//
// What bounded them: in general_kernel every wave loads, writes LDS, reads fragments and multiplies,
// all in step, so the vector memory path, the LDS and the matrix pipe follow one another (NT bf16
// 1000 x 2003 x 1500: 24 steps of 1,250 cycles of which the matrix pipe needs 256).  Here the
// loading waves keep DEPTH sub-blocks in flight in registers and write the next one into the other
// of two LDS stages while the multiplying waves, one per SIMD, read and multiply this one, each
// half's reads under the other half's instructions.  One barrier per sub-block.
// Eight loading waves where no second workgroup shares the CU: a CU takes 57 B/ns of four waves'
// loads, 77-96 of eight (128 x 64 tile above: 18.8 us undivided, 17.0 with four, 15.9 with eight).
// fp32 is bound by its matrix instruction, and four are enough.  Measured before -> now (us):
// fp32 777 x 1001 x 1301 NT 32.3 -> 25.6 (20 of it the matrix pipe of 208 tiles), NN 38.7 -> 31.3, 2001^3 NT
// 142 -> 128; bf16 1000 x 2003 x 1500 NN 22.4 -> 18.5, TN 23.3 -> 20.2;
// int8 1000 x 2003 x 1500 NN 15.8 -> 12.4; FP8 2000^3 NT 29.4 -> 23.6.
// What bounds the 16-bit tiles now: the loads of rows that start off 16 bytes (1000 x 2003 x 1500 NT: 24 KiB per step of
// 0.335 us, 72 B/ns).
#pragma once

namespace brg {

// One operand of the loading waves.
template <int KIND, int EXT, bool KMAJ, int GT>
struct DutyLoader : GenLoader<KIND, EXT, KMAJ, EXT * 8 / GT, GT, ROWS_NEAR> {
    typedef GenLoader<KIND, EXT, KMAJ, EXT * 8 / GT, GT, ROWS_NEAR> Base;
    static constexpr int CH = EXT * 8 / GT;
    int over;                   // elements by which this thread's chunks were moved back at an edge (the same for all:
                                // GT threads take whole k-rows)

    __device__ void init(int tg, int64_t first, int64_t limit, int64_t ld, int64_t K, bool packed)
    {
        Base::init(tg, first, limit, ld, K, packed);
        over = 0;
        if constexpr (!KMAJ) {
            const int64_t o = first + (int64_t)(tg % Base::Img::CPR) * Base::E - (limit - Base::E);
            over = o <= 0 ? 0 : o < Base::E ? (int)o : Base::E;
        }
    }
    // Step 0 of the problem, which is its incomplete sub-block `kb` when `tail`: read like any
    // chunk that would run past the end of its run (a k-contiguous one from the run's last 16 bytes,
    // an m/n-contiguous one in the last k-row), `short_by` elements of it shifted out or all of it zero.
    __device__ __forceinline__ void load_first(const char *base, int64_t kb, bool tail, typename Base::Raw (&raw)[CH]) const
    {
        const char *b = base + Base::origin;
        if constexpr (KMAJ) {
            const int64_t back = tail ? (int64_t)short_by(kb, tail) * Base::S : 0;
#pragma unroll
            for (int j = 0; j < CH; ++j)
                raw[j] = gen_load<KIND>(b - back + Base::rel[j]);
        } else {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int64_t past = kb * Base::SUB + k_row(j) - (Base::K - 1);
                raw[j] = gen_load<KIND>(b - (tail && past > 0 ? past * Base::ld * Base::S : 0) + Base::rel[j]);
            }
        }
    }
    __device__ __forceinline__ int k_row(int j) const { return (j * GT + Base::tg) / Base::Img::CPR; }
    __device__ __forceinline__ int64_t short_by(int64_t kb, bool tail) const
    {
        const int64_t past = kb * Base::SUB + (Base::tg & 7) * Base::E - (Base::K - Base::E);
        return tail && past > 0 ? past : 0;
    }
    __device__ __forceinline__ void finish_first(LDS_AS char *img, int64_t kb, bool tail, const typename Base::Raw (&raw)[CH]) const
    {
        int n = over;
        if constexpr (KMAJ) {
            const int64_t by = short_by(kb, tail);
            n = by < Base::E ? (int)by : Base::E;
        }
        asm volatile("" : "+v"(n));
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            typename Base::Raw v = gen_shift<KIND>(raw[j], n);
            if (!KMAJ && tail && kb * Base::SUB + k_row(j) >= Base::K)
                v = typename Base::Raw{};
            *(LDS_AS gu32x4 *)(img + Base::Img::dst_byte(j * GT + Base::tg)) = gen_to_lds<KIND>(v);
        }
    }
    // At an edge: with what was moved back shifted out.  (The count is kept from the compiler, which
    // would hold every mask and selection it leads to in registers across the loop.)
    __device__ __forceinline__ void finish_edge(LDS_AS char *img, const typename Base::Raw (&raw)[CH]) const
    {
        int n = over;
        asm volatile("" : "+v"(n));
#pragma unroll
        for (int j = 0; j < CH; ++j)
            *(LDS_AS gu32x4 *)(img + Base::Img::dst_byte(j * GT + Base::tg)) =
                gen_to_lds<KIND>(KMAJ ? raw[j] : gen_shift<KIND>(raw[j], n));
    }
    // `base`: the matrix plus the sub-block's step
    __device__ __forceinline__ void load_at(const char *base, typename Base::Raw (&raw)[CH]) const
    {
        // (both opaque to the compiler, which would keep a 64-bit address per load across the loop)
        const GLB_AS char *b = (const GLB_AS char *)uniform_ptr((const uint16_t *)(base + Base::origin));
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            uint32_t o = Base::rel[j];
            asm volatile("" : "+v"(o));
            raw[j] = Base::load_from(b, o);
        }
        __builtin_amdgcn_sched_barrier(0);          // in the order in which they are waited for
    }
};

// How a multiplying wave adds up.  One chain of fp32 additions over all of K is further from the
// exact sum than the two or more chains of the undivided tiles and of split reductions, so a 64 x 64 tile has
// kChains sets of accumulators, and every kEvery sub-blocks what the accumulators hold is added to
// totals (closed off) and they start again from zero.  Not where the sum becomes 16 bits, which hide it, and integers
// are exact.  The totals stay in LDS where registers for them would cost a workgroup: the 16-bit 128 x 128 tile has none left, and the
// 64 x 64 tile with both operands along k (76 registers) runs three to a CU, in registers (89) two: fp32 3950 x 721 x 161
// 16.6 us, 18.1; FP8 1232 x 1696 x 257 9.8, 11.5 (so FP8 has the two chains alone).  For one-byte operands, converted by
// the loading waves, the wider tiles have none.  Error relative to one chain: 16-bit 64 x 64, 128 x 64 and 128 x 128 0.64, 0.55 and 0.85, fp32
// 64 x 64 0.70 (23,000 drawn products); fp32 128 x 64 and 128 x 128 0.74 and 0.85 (500; closed off every fourth sub-block 0.4, at 4 to 5 % of the
// time: 1904 x 9008 x 1089 309 us, 326).  Time within 1 % on average, the 16-bit 128 x 128 tile with both operands along m and n 5 %.
enum { TOTALS_NONE, TOTALS_REGS, TOTALS_LDS };
template <int KIND, int BM, int BN>
struct DutySums {
    static constexpr bool F32 = KIND == KIND_F32, WIDE = BM * BN == 128 * 128, NARROW = BM * BN == 64 * 64;
    static constexpr int kChains = KIND == KIND_S8 || !NARROW ? 1 : 2;      // one for each half of a sub-block
    static constexpr int kTotals = kind_is_8bit(KIND) ? TOTALS_NONE : NARROW || (!F32 && WIDE) ? TOTALS_LDS : TOTALS_REGS;
    static constexpr int kEvery = F32 ? (NARROW ? 32 : 16) : NARROW || WIDE ? 16 : 8;
};

template <int KIND, int BM, int BN>
struct DutyConfig {
    static constexpr uint32_t STAGE = (BM + BN) * 128;      // LDS bytes of one sub-block
    static constexpr int EPI_LD = BN + 4;
    // Totals in LDS come behind both the stages and the staged result: a wave may stage its sums while another's
    // last reads of its totals are under way.
    static constexpr size_t kTotalsAt = 2 * (size_t)STAGE > (size_t)BM * EPI_LD * 4 ? 2 * (size_t)STAGE : (size_t)BM * EPI_LD * 4;
    static constexpr size_t kLds = kTotalsAt + (DutySums<KIND, BM, BN>::kTotals == TOTALS_LDS ? (size_t)BM * BN * 4 : 0);
    static_assert(kTotalsAt % 1024 == 0 && kLds <= 160 * 1024, "");
};

template <int MODE, int R, int TILES>
struct DutyTotals {
    typedef float Vec __attribute__((ext_vector_type(R)));
    Vec total[MODE == TOTALS_REGS ? TILES : 1];
    LDS_AS Vec *mine;           // TOTALS_LDS: this lane's of accumulator 0, those of the next 64 further on
    bool any;                   // ... are there

    __device__ __forceinline__ void begin(LDS_AS char *room, int lane)
    {
        mine = (LDS_AS Vec *)room + lane;
        any = false;
    }
    __device__ __forceinline__ void add(int i, const Vec &sum)
    {
        if constexpr (MODE == TOTALS_LDS)
            mine[i * 64] = any ? mine[i * 64] + sum : sum;
        else
            total[i] = any ? total[i] + sum : sum;
    }
    __device__ __forceinline__ Vec with(int i, const Vec &sum) const
    {
        if constexpr (MODE == TOTALS_LDS)
            return any ? mine[i * 64] + sum : sum;
        else
            return MODE == TOTALS_REGS && any ? total[i] + sum : sum;
    }
};

template <int KIND, bool A_KMAJ, bool B_KMAJ, int BM, int BN, int NLW, int DEPTH, int PER_CU>
__global__ void __launch_bounds__((4 + NLW) * 64, (4 + NLW) / 4 * PER_CU)
general_duty_kernel(GenArgs p)
{
    typedef DutyConfig<KIND, BM, BN> Cfg;
    constexpr bool F32 = KIND == KIND_F32;
    constexpr int MT = F32 ? 32 : 16;
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / MT, TN = WN / MT;
    typedef DutySums<KIND, BM, BN> Sums;
    constexpr int CHAINS = Sums::kChains;
    typedef DutyLoader<KIND, BM, A_KMAJ, NLW * 64> LoadA;
    typedef DutyLoader<KIND, BN, B_KMAJ, NLW * 64> LoadB;
    typedef typename LoadA::Img ImgA;
    typedef typename LoadB::Img ImgB;
    constexpr int S = GenElem<KIND>::S, SUB = GenElem<KIND>::SUB;

    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    LDS_AS char *smem = (LDS_AS char *)smem_generic;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int64_t z = blockIdx.z;
    const char *Abase = p.A + z * p.ms_a * S, *Bbase = p.B + z * p.ms_b * S;
    p.epi.C = (char *)p.epi.C + z * p.ms_c * (p.epi.c_f32 ? 4 : 2);

    int tile, slice, tm, tn;
    slice_major_coords(p.tiles_m * p.tiles_n, p.split, p.walk, tile, slice);
    group_walk(tile, p.tiles_m, p.tiles_n, p.walk, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    const int total = (int)((p.K + SUB - 1) / SUB);
    const int per = (int)p.walk.per;
    const int begin = slice * per < total ? slice * per : total;
    const int end = begin + per < total ? begin + per : total;
    const int n = end - begin;

    if (w >= 4) {
        // ---------------- loader waves ----------------
        const int tg = tid - 256;
        LoadA la;
        LoadB lb;
        la.init(tg, m0, p.M, p.lda, p.K, false);
        lb.init(tg, n0, p.N, p.ldb, p.K, p.b_packed != 0);
        struct Set {
            typename LoadA::Raw a[LoadA::CH];
            typename LoadB::Raw b[LoadB::CH];
        };
        // An incomplete sub-block (the K tail) is taken first: step 0 stands for it, step u
        // for sub-block u - 1.  The cursor stops at the last step, which is then repeated.
        const bool ragged = p.K % SUB != 0;
        int u = begin < total ? begin : total - 1;
        const bool tail = ragged && u == 0;
        const int rot = ragged ? 1 : 0;
        auto run = [&](auto edges) {
            constexpr bool EDGES = decltype(edges)::value;
            Set sets[DEPTH];
            auto issue = [&](Set &s) {
                const int at = u - rot > 0 ? u - rot : 0;
                la.load_at(Abase + at * la.step, s.a);
                lb.load_at(Bbase + at * lb.step, s.b);
                u = u + 1 < total ? u + 1 : u;
            };
            auto finish = [&](const Set &s, int stage) {
                LDS_AS char *at = smem + (uint32_t)stage * Cfg::STAGE;
                if constexpr (EDGES) {
                    la.finish_edge(at, s.a);
                    lb.finish_edge(at + ImgA::BYTES, s.b);
                } else {
                    la.finish_whole(at, s.a);
                    lb.finish_whole(at + ImgA::BYTES, s.b);
                }
            };
            const int64_t at0 = tail ? total - 1 : u - rot;
            // (an incomplete or an edge's; a whole sub-block needs none of what that does)
            if (EDGES || tail) {
                la.load_first(Abase + at0 * la.step, at0, tail, sets[0].a);
                lb.load_first(Bbase + at0 * lb.step, at0, tail && !lb.packed, sets[0].b);
            } else {
                la.load_at(Abase + at0 * la.step, sets[0].a);
                lb.load_at(Bbase + at0 * lb.step, sets[0].b);
            }
            u = u + 1 < total ? u + 1 : u;
            static_for<1, DEPTH>([&](auto d) { issue(sets[decltype(d)::value]); });
            if (EDGES || tail) {
                la.finish_first(smem, at0, tail, sets[0].a);
                lb.finish_first(smem + ImgA::BYTES, at0, tail && !lb.packed, sets[0].b);
            } else {
                finish(sets[0], 0);
            }
            issue(sets[0]);
            wait_lgkmcnt0();
            if (n > 0)
                block_sync();                       // B(0)
            auto step = [&](int t, Set &s) {
                finish(s, t & 1);                   // step t, into the stage that step t - 2 has left
                issue(s);                           // step t + DEPTH
                wait_lgkmcnt0();
                block_sync();                       // B(t)
            };
            // Whole turns of the sets, then the rest: with a way out of the middle of a turn the
            // compiler, which merges what is in flight on every way, would wait for all of it.
            int t = 1;
            for (; t + DEPTH <= n; t += DEPTH)
                static_for<0, DEPTH>([&](auto d) { step(t + decltype(d)::value, sets[(decltype(d)::value + 1) % DEPTH]); });
            static_for<0, DEPTH - 1>([&](auto d) {
                if (t + decltype(d)::value < n)
                    step(t + decltype(d)::value, sets[(decltype(d)::value + 1) % DEPTH]);
            });
        };
        if (la.edge || lb.edge)
            run(std::true_type{});
        else
            run(std::false_type{});
        block_sync();                               // E1
        block_sync();                               // E2: the staged tile is complete
        if (NLW > 4 && w >= 8)
            return;                                 // eight waves store
    } else {
        // ---------------- multiplying waves ----------------
        const int wm = w >> 1, wn = w & 1;
        typedef std::conditional_t<F32, f32x16, f32x4> Acc;
        Acc acc[CHAINS][TN][TM];
#pragma unroll
        for (int c = 0; c < CHAINS; ++c)
#pragma unroll
            for (int a = 0; a < TN; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[c][a][b] = 0.0f;
        DutyTotals<Sums::kTotals, F32 ? 16 : 4, TN * TM> totals;
        totals.begin(smem + Cfg::kTotalsAt + w * (TN * TM * (F32 ? 4096 : 1024)), lane);
        // (a 16-bit C hides what the totals would add)
        const bool with_totals = Sums::kTotals != TOTALS_NONE && (F32 || p.split > 1 || p.epi.c_f32);
        bf16x8 fa16[2][F32 ? 1 : TM], fb16[2][F32 ? 1 : TN];
        f32x4 fa32[2][2][F32 ? TM : 1], fb32[2][2][F32 ? TN : 1];
        auto read_half = [&](LDS_AS char *at, auto hc) {
            constexpr int h = decltype(hc)::value;
            LDS_AS char *bt = at + ImgA::BYTES;
            if constexpr (F32) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
#pragma unroll
                    for (int t = 0; t < TM; ++t)
                        fa32[h][j][t] = ImgA::frag32(at, wm * WM, t, 2 * h + j, lane);
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        fb32[h][j][t] = ImgB::frag32(bt, wn * WN, t, 2 * h + j, lane);
                }
            } else {
#pragma unroll
                for (int t = 0; t < TM; ++t)
                    fa16[h][t] = ImgA::frag16(at, wm * WM, t, h, lane);
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    fb16[h][t] = ImgB::frag16(bt, wn * WN, t, h, lane);
            }
        };
        auto multiply_half = [&](auto hc) {
            constexpr int h = decltype(hc)::value, c = h % CHAINS;
            if constexpr (F32) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int a = 0; a < TN; ++a)
#pragma unroll
                            for (int b = 0; b < TM; ++b)
                                acc[c][a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb32[h][j][a][e], fa32[h][j][b][e],
                                                                                   acc[c][a][b], 0, 0, 0);
            } else {
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b)
                        acc[c][a][b] = mfma_16x16x32<kind_is_f8(KIND) ? KIND_BF16 : KIND>(fb16[h][a], fa16[h][b], acc[c][a][b]);
            }
        };
        auto chains = [&](int a, int b) {
            if constexpr (CHAINS == 2)
                return acc[0][a][b] + acc[1][a][b];
            else
                return acc[0][a][b];
        };
        constexpr std::integral_constant<int, 0> H0{};
        constexpr std::integral_constant<int, 1> H1{};
        for (int t = 0; t < n; ++t) {
            block_sync();                           // B(t): step t is in LDS
            LDS_AS char *at = smem + (uint32_t)(t & 1) * Cfg::STAGE;
            read_half(at, H0);
            if (t > 0)
                multiply_half(H1);                  // second half of step t - 1
            if (with_totals && t > 0 && t % Sums::kEvery == 0) {
                asm volatile("");                   // (a branch: selected by step, this took 22 % of the fp32 64 x 64 tile's time)
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b) {
                        totals.add(a * TM + b, chains(a, b));
#pragma unroll
                        for (int c = 0; c < CHAINS; ++c)
                            acc[c][a][b] = 0.0f;
                    }
                totals.any = true;
            }
            __builtin_amdgcn_sched_barrier(0);
            read_half(at, H1);
            multiply_half(H0);
            __builtin_amdgcn_sched_barrier(0);
            wait_lgkmcnt0();                        // every read of step t is complete before B(t + 1)
        }
        if (n > 0)
            multiply_half(H1);
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[0][a][b] = totals.with(a * TM + b, chains(a, b));
        block_sync();                               // E1: nobody reads fragments any more
        LDS_AS float *stage = (LDS_AS float *)smem;
        static_for<0, TN * TM>([&](auto ic) {
            constexpr int a = decltype(ic)::value / TM, b = decltype(ic)::value % TM;
            if constexpr (F32) {
                static_for<0, 4>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    const Acc &v = acc[0][a][b];
                    *(LDS_AS f32x4 *)(stage + (wm * WM + 32 * b + (lane & 31)) * Cfg::EPI_LD + wn * WN + 32 * a + 8 * q + 4 * (lane >> 5)) =
                        f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                });
            } else {
                *(LDS_AS f32x4 *)(stage + (wm * WM + 16 * b + (lane & 15)) * Cfg::EPI_LD + wn * WN + 16 * a + 4 * (lane >> 4)) =
                    acc[0][a][b];
            }
        });
        wait_lgkmcnt0();
        block_sync();                               // E2
    }
    gen_store_sums<KIND, BM, BN, 512, 1, true>(p, smem, tid, m0, n0, slice);
}

template <int KIND, bool A_KMAJ, bool B_KMAJ, int BM, int BN, int NLW, int DEPTH, int PER_CU>
hipError_t duty_launch(const Problem &p)
{
    typedef DutyConfig<KIND, BM, BN> Cfg;
    GenArgs a = gen_args(p);
    a.tiles_m = (int)((p.M + BM - 1) / BM);
    a.tiles_n = (int)((p.N + BN - 1) / BN);
    a.walk = make_walk(a.tiles_m, a.tiles_n, p.split, (p.K + GenElem<KIND>::SUB - 1) / GenElem<KIND>::SUB, 1, (int64_t)kWalkRows * a.tiles_n);
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)p.split, (unsigned)p.nmat);
    void (*kern)(GenArgs) = general_duty_kernel<KIND, A_KMAJ, B_KMAJ, BM, BN, NLW, DEPTH, PER_CU>;
    static thread_local bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Cfg::kLds);
        if (e != hipSuccess)
            return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3((4 + NLW) * 64), Cfg::kLds, p.stream, a);
    return hipGetLastError();
}

// Which tiles of an eligible problem the divided kernel takes: the others run undivided, where the deeper start is not
// paid back (the 32 x 32 tile's groups of one wave have no barrier to wait at).  Times divided / undivided below are
// means over 3,200 problems of 4 to 60 sub-blocks in four layouts, on 16-byte rows and off them.
inline bool duty_runs(const Problem &p, int tile)
{
    if (tile == GEN_32 || !duty_eligible(p))
        return false;
    const int64_t bn = tile == GEN_128 ? 128 : 64, bm = tile == GEN_64 ? 64 : 128;
    const int64_t tiles = ((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn), wgs = tiles * p.split * p.nmat;
    if (tiles * 768 > 0xffffffffLL)                 // (the host cuts such problems first)
        return false;
    const int64_t sub = p.in_s8 ? 128 : (in_16bit(p) || in_8bit(p)) ? 64 : 32, steps = (p.K + sub - 1) / sub / p.split;
    const int k_rows = (p.transA == 0) + (p.transB == 1);       // operands stored along k
    if (tile == GEN_128) {
        // Beyond one round two undivided workgroups of a CU overlap as much (bf16 NT 3001^3 105 against 110-118 us); fp32
        // 1.03 to 1.10 with up to 8 sub-blocks, 1.00 to 1.02 with 9 to 14, 0.95 to 0.97 with more (2228 x 6534 x 115 TT 52.7 undivided, 60.9).
        return wgs <= 256 || (!in_16bit(p) && !in_8bit(p) && steps >= 12);
    }
    if (p.in_s8) {
        // Both operands along k: 1.05 to 1.08 with fewer than 15 sub-blocks and 1.01 to 1.03 with more, on 4-byte rows 0.86 to 0.99;
        // both along m and n, 64 x 64: 1.02 to 1.08, 1.00, on 16-byte rows 0.99; else 0.77 to 0.98 (128 x 64 beyond a round: 3000^3 60 us undivided, 67).
        const uintptr_t at = (uintptr_t)p.A | (uintptr_t)p.B | (uintptr_t)p.lda | (uintptr_t)p.ldb;
        if (tile == GEN_MID)
            return wgs <= 256 && (k_rows < 2 || !(at & 3));
        return k_rows == 1 || steps >= 15 || !(at & (k_rows == 2 ? 3 : 15));
    }
    // FP8's 128 x 64 has registers for one workgroup on a CU: beyond a round 1.26 with up to 8 sub-blocks (NN and TN, more than two rounds:
    // 1.28), 0.88 to 0.99 with 15 and more within two rounds, 0.90 to 1.03 with both operands along k.
    if (tile == GEN_MID && in_8bit(p))
        return wgs <= 256 || (wgs <= 512 && (k_rows == 2 || steps >= 15)) || (k_rows == 2 && steps >= 9);
    return true;
}

template <int KIND, bool A_KMAJ, bool B_KMAJ>
hipError_t duty_tile(const Problem &p, int tile)
{
    if constexpr (KIND == KIND_F32) {
        switch (tile) {
        case GEN_128: return duty_launch<KIND, A_KMAJ, B_KMAJ, 128, 128, 4, 4, 1>(p);
        case GEN_MID: return duty_launch<KIND, A_KMAJ, B_KMAJ, 128, 64, 4, 3, 2>(p);
        default: return duty_launch<KIND, A_KMAJ, B_KMAJ, 64, 64, 4, 4, 2>(p);
        }
    } else {
        switch (tile) {
        case GEN_128: return duty_launch<KIND, A_KMAJ, B_KMAJ, 128, 128, 8, 4, 1>(p);
        case GEN_MID:
            // (one-byte operands: no registers for two workgroups of it on a CU, FP8 3000^3 85 us with one)
            if constexpr (!kind_is_8bit(KIND)) {
                if (((p.M + 127) / 128) * ((p.N + 63) / 64) * p.split * p.nmat > 256)
                    return duty_launch<KIND, A_KMAJ, B_KMAJ, 128, 64, 4, 3, 2>(p);
            }
            return duty_launch<KIND, A_KMAJ, B_KMAJ, 128, 64, 8, 5, 1>(p);
        default: return duty_launch<KIND, A_KMAJ, B_KMAJ, 64, 64, 4, 4, 2>(p);
        }
    }
}

}  // namespace brg
