// General GEMM / batch-reduce kernel for gfx950: any M, N, K, batch, leading dimensions,
// alignment and transpose flags, on the matrix instructions of the operands' own type.
// It takes every problem the alignment rules of the tuned kernels turn away, and the
// small fp32 grids that 128 x 128 tiles leave most of the chip idle on.
//
// Structure (Algorithm 1 of the paper, mapped to a GPU): one workgroup owns a BM x BN
// block of C; the reduction is cut into sub-blocks of 128 bytes of k (64 16-bit, 128
// int8, 32 fp32 values; an FP8 operand is widened exactly to bf16 on the way into LDS,
// 64 values) which are dealt round-robin to KW groups of WGM x WGN wavefronts.  Every
// group keeps a whole BM x BN accumulator tile in registers over its share of the batch
// and K loops (Section 2.1, advantage (1)); the KW tiles are added in a fixed order
// through LDS at the end, where beta / bias / ReLU / narrowing are applied once.
//
// What bounds it: operands that are not 16-byte aligned cannot use the global->LDS DMA,
// so every byte passes through registers (global load, LDS write, LDS read).  The load
// of a sub-block is therefore issued one or two steps ahead into registers, and written to
// the other of two LDS stages before the current one is multiplied.  (The wide tiles divide this
// between waves where the reduction is long enough: general_duty.hpp.)  What a ragged
// edge needs is decided per 16-byte chunk, not per element: a chunk that would run past
// the end of its run (the K tail of a k-contiguous operand, the last columns of an
// m/n-contiguous one) is read as the run's LAST 16 bytes and shifted down in registers,
// which fills with zeros - one load, always inside the matrix, at any alignment.  A CU
// takes 70-110 B/ns of 16-byte loads from 16-byte aligned rows, 80 from dword-aligned
// ones, 53 where every second row starts at an odd 2-byte address and 35 where all do.
// (Before: element by element with bounds checks into the fp32 instruction.  NT bf16
// 1000 x 2003 x 1500 315 -> 20.1 us, NT fp32 777 x 1001 x 1301 216 -> 33.6 us.)
#pragma once
#include "bf16_tiles.hpp"

namespace brg {

struct GenArgs {
    int64_t M, N, K, batch;
    const char *A;
    const int64_t *A_off;
    int64_t lda;
    const char *B;
    const int64_t *B_off;
    int64_t ldb;
    int b_packed;
    Epilogue epi;
    int split;
    float *partial;
    int tiles_m, tiles_n;
    Walk walk;
    int64_t ms_a, ms_b, ms_c;       // element strides between the matrices of a batched call
};

// Element facts per operand kind: bytes in memory, elements per 16-byte LDS chunk, k per
// 128-byte sub-block.
template <int KIND>
struct GenElem {
    static constexpr int S = KIND == KIND_F32 ? 4 : kind_is_8bit(KIND) ? 1 : 2;
    static constexpr int E = KIND == KIND_F32 ? 4 : KIND == KIND_S8 ? 16 : 8;
    static constexpr int SUB = 8 * E;
};

// A chunk as it comes from memory: E * S bytes, 16 (FP8: 8).
template <int KIND>
struct GenRawOf { typedef std::conditional_t<kind_is_f8(KIND), gu32x2, gu32x4> type; };

// The loads are one instruction at any alignment (the hardware takes unaligned global
// accesses); the typedefs tell the compiler no more than the element's own alignment.
typedef uint32_t u32x2_any1 __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_any1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x4_any2 __attribute__((ext_vector_type(4), aligned(2)));

template <int KIND>
__device__ __forceinline__ typename GenRawOf<KIND>::type gen_load(const char *p)
{
    if constexpr (kind_is_f8(KIND))
        return *(const u32x2_any1 *)p;
    else if constexpr (KIND == KIND_F32)
        return *(const u32x4_any4 *)p;
    else if constexpr (KIND == KIND_S8)
        return *(const u32x4_any1 *)p;
    else
        return *(const u32x4_any2 *)p;
}

// A chunk in memory, at the element's own alignment.
template <int KIND>
struct GenAnyOf {
    typedef std::conditional_t<kind_is_f8(KIND), u32x2_any1,
            std::conditional_t<KIND == KIND_F32, u32x4_any4, std::conditional_t<KIND == KIND_S8, u32x4_any1, u32x4_any2>>> type;
};

// Drop the first `n` elements and fill with zeros from the top (n = E: all zero), without
// branches: whole words by halving selects, the rest by v_alignbyte.
template <int KIND>
__device__ __forceinline__ typename GenRawOf<KIND>::type gen_shift(typename GenRawOf<KIND>::type v, int n)
{
    constexpr int W = kind_is_f8(KIND) ? 2 : 4;
    const uint32_t bytes = (uint32_t)n * GenElem<KIND>::S, words = bytes >> 2;
    uint32_t w[W + 1];
#pragma unroll
    for (int i = 0; i < W; ++i)
        w[i] = v[i];
    w[W] = 0;
#pragma unroll
    for (int by = 1; by <= W; by *= 2) {
#pragma unroll
        for (int i = 0; i < W; ++i)
            w[i] = (words & by) ? (i + by < W ? w[i + by] : 0u) : w[i];
    }
#pragma unroll
    for (int i = 0; i < W; ++i)
        v[i] = GenElem<KIND>::S == 4 ? w[i] : __builtin_amdgcn_alignbyte(w[i + 1], w[i], bytes & 3u);
    return v;
}

// Chunk of a run shorter than a chunk: element e comes from p + e while e < count.
template <int KIND>
__device__ __forceinline__ typename GenRawOf<KIND>::type gen_gather(const char *p, int64_t count)
{
    constexpr int S = GenElem<KIND>::S, E = GenElem<KIND>::E;
    typename GenRawOf<KIND>::type v = {};
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < count) {
            uint32_t x;
            if constexpr (S == 4)
                x = ((const uint32_t *)p)[e];
            else if constexpr (S == 2)
                x = ((const uint16_t *)p)[e];
            else
                x = ((const uint8_t *)p)[e];
            v[e * S / 4] |= x << (8 * (e * S % 4));
        }
    }
    return v;
}

// What goes into LDS: the bytes themselves, or eight FP8 values widened exactly to bf16
// (their 2 or 3 fraction bits and exponent range fit; NaN and infinities stay).
template <int KIND>
__device__ __forceinline__ gu32x4 gen_to_lds(typename GenRawOf<KIND>::type v)
{
    if constexpr (kind_is_f8(KIND)) {
        typedef __attribute__((ext_vector_type(2))) float f32x2_t;
        gu32x4 r;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x2_t a, b;
            if constexpr (KIND == KIND_BF8) {
                a = __builtin_amdgcn_cvt_pk_f32_bf8((int)v[h], false);
                b = __builtin_amdgcn_cvt_pk_f32_bf8((int)v[h], true);
            } else {
                a = __builtin_amdgcn_cvt_pk_f32_fp8((int)v[h], false);
                b = __builtin_amdgcn_cvt_pk_f32_fp8((int)v[h], true);
            }
            r[2 * h] = pack_bf16x2(a[0], a[1]);
            r[2 * h + 1] = pack_bf16x2(b[0], b[1]);
        }
        return r;
    } else {
        return v;
    }
}

// LDS image of one operand sub-block: EXT rows / columns of m or n by 128 bytes of k.
// k-contiguous operands: 128-byte rows, chunk c of row r at c ^ ((r >> 1) & 7).
// m/n-contiguous operands: k-rows of EXT elements; the chunk swizzles below give the rows
// that one transposing (16-bit, int8) or 32-bit (fp32) read of a half-wave touches
// different places of the 256-byte bank window, for every row length.
template <int KIND, int EXT, bool KMAJ>
struct GenImage {
    static constexpr int E = GenElem<KIND>::E;
    static constexpr int CPR = EXT / E;                 // chunks per k-row (m/n-contiguous)
    static constexpr int ROWB = CPR * 16;
    static constexpr uint32_t BYTES = EXT * 128;

    __device__ static int swz(int kr)
    {
        if constexpr (KIND == KIND_F32)
            return EXT >= 64 ? ((kr >> 2) & 1) << 3 : 0;
        else if constexpr (KIND == KIND_S8)
            return EXT >= 128 ? (((kr >> 1) & 3) | (((kr >> 4) & 1) << 2))
                   : EXT == 64 ? (((kr >> 2) & 1) | (((kr >> 4) & 1) << 1)) : ((kr >> 4) & 1);
        else
            return EXT >= 128 ? (((kr & 3) << 2) | (((kr >> 3) & 1) << 1))
                   : EXT == 64 ? ((((kr >> 1) & 1) << 1) | (((kr >> 3) & 1) << 2)) : (((kr >> 3) & 1) << 1);
    }
    // 128-byte fp32 k-rows (EXT = 32): rows kr and kr + 4, read together, go to different
    // halves of the bank window by exchanging neighbouring rows.
    __device__ static int row_place(int kr) { return KIND == KIND_F32 && EXT == 32 ? kr ^ ((kr >> 2) & 1) : kr; }

    __device__ static uint32_t dst_byte(int idx)
    {
        if constexpr (KMAJ) {
            const int r = idx >> 3, c = idx & 7;
            return (uint32_t)(r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
        } else {
            const int kr = idx / CPR, c = idx % CPR;
            return (uint32_t)(row_place(kr) * ROWB + ((c ^ swz(kr)) << 4));
        }
    }
    // Operand of the 16x16 instructions for 16-row tile t and half s of the sub-block.
    __device__ static bf16x8 frag16(LDS_AS char *img, int base, int t, int s, int lane)
    {
        if constexpr (KMAJ) {
            const int r = base + t * 16 + (lane & 15);
            const int c = 4 * s + (lane >> 4);
            return *(LDS_AS bf16x8 *)(img + (uint32_t)(r * 128 + ((c ^ ((r >> 1) & 7)) << 4)));
        } else if constexpr (KIND == KIND_S8) {
            const int i = lane & 15, c = (base + t * 16) >> 4;
            i32x2 v[2];
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) {
                const int kr = 64 * s + 16 * (lane >> 4) + 8 * rd + (i >> 1);
                v[rd] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                    (LDS_AS i32x2 *)(img + (uint32_t)(kr * ROWB + ((c ^ swz(kr)) << 4) + 8 * (i & 1))));
            }
            return __builtin_bit_cast(bf16x8, (i32x4)__builtin_shufflevector(v[0], v[1], 0, 1, 2, 3));
        } else {
            const int b = lane >> 4, i = lane & 15;
            const int col = base + t * 16 + 4 * (i & 3);
            s16x4 v[2];
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) {
                const int kr = s * 32 + 8 * b + 4 * rd + (i >> 2);
                v[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (LDS_AS s16x4 *)(img + (uint32_t)(kr * ROWB + (((col >> 3) ^ swz(kr)) << 4) + (col & 7) * 2)));
            }
            return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
    // fp32: the four k = 8j + 4*(lane/32) + 0..3 of row t*32 + lane%32 (the k order inside
    // an instruction is free as long as both operands agree).
    __device__ static f32x4 frag32(LDS_AS char *img, int base, int t, int j, int lane)
    {
        const int h = lane >> 5;
        const int r = base + t * 32 + (lane & 31);
        if constexpr (KMAJ) {
            const int c = 2 * j + h;
            return *(LDS_AS f32x4 *)(img + (uint32_t)(r * 128 + ((c ^ ((r >> 1) & 7)) << 4)));
        } else {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int kr = 8 * j + 4 * h + e;
                v[e] = *(LDS_AS float *)(img + (uint32_t)(row_place(kr) * ROWB + (((r >> 2) ^ swz(kr)) << 4) + (r & 3) * 4));
            }
            return v;
        }
    }
};

// One operand of one wave group: where its CH chunks per thread come from.  `first` /
// `limit`: first row or column of the tile and the matrix extent in that direction.
// A chunk's place is an offset from `origin`, which is the same for all lanes: 32 bits (general_offsets_fit says which
// problems they hold), so that a load is one instruction on a scalar base; 64 for runs too short for that and rows too far apart.
enum RowsAre { ROWS_NEAR, ROWS_SHORT, ROWS_FAR };
template <int KIND, int EXT, bool KMAJ, int CH, int GT, int ROWS>
struct GenLoader {
    typedef GenImage<KIND, EXT, KMAJ> Img;
    typedef typename GenRawOf<KIND>::type Raw;
    static constexpr bool TINY = ROWS == ROWS_SHORT;
    typedef std::conditional_t<ROWS == ROWS_NEAR, uint32_t, int64_t> Off;
    static constexpr int S = GenElem<KIND>::S, E = GenElem<KIND>::E, SUB = GenElem<KIND>::SUB;
    static_assert(GT % 8 == 0 && GT % Img::CPR == 0, "a thread's chunks share their place along a row");
    Off rel[CH];                // bytes from the tile's origin, sub-block 0
    int64_t origin;             // bytes from the matrix to it
    int64_t ld, K, step, run;   // step: bytes per sub-block; run: elements of a contiguous run
    int64_t first, limit;
    bool packed, edge, tiny;
    int tg;

    __device__ void init(int tg_, int64_t first_, int64_t limit_, int64_t ld_, int64_t K_, bool packed_)
    {
        tg = tg_; first = first_; limit = limit_; ld = ld_; K = K_; packed = KMAJ && packed_;
        run = KMAJ ? K : limit;
        // (With whole chunks the ones beyond the limit only repeat the last: nobody stores them.)
        edge = !KMAJ && first + EXT > limit && limit % E != 0;
        tiny = TINY && !packed && run < E;
        step = KMAJ ? (packed ? 8 * ld * S : (int64_t)SUB * S) : (int64_t)SUB * ld * S;
        if constexpr (KMAJ) {
            const Off ldo = (Off)ld * (Off)S, c = (Off)(tg & 7);
            const int last = (int)(limit - 1 - first < EXT ? limit - 1 - first : EXT);      // rows past it repeat it
            origin = (packed ? first * 8 : first * ld) * S;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int r = (j * GT + tg) >> 3;
                rel[j] = packed ? c * ldo + (Off)(r * 8 * S) : (Off)(r < last ? r : last) * ldo + c * (Off)(E * S);
            }
        } else {
            // (columns past the last whole chunk repeat it)
            const int64_t far = limit - E > 0 ? limit - E : 0;
            const int64_t base = tiny || first < far ? first : far;
            const int col = tg % Img::CPR * E, room = (int)(far - base < EXT ? far - base : EXT);
            const Off at = (Off)((tiny || col < room ? col : room) * S), ldo = (Off)ld * (Off)S;
            origin = base * S;
#pragma unroll
            for (int j = 0; j < CH; ++j)
                rel[j] = (Off)((j * GT + tg) / Img::CPR) * ldo + at;
        }
    }
    __device__ __forceinline__ static Raw load_from(const GLB_AS char *base, Off off)
    {
        return *(const GLB_AS typename GenAnyOf<KIND>::type *)(base + off);
    }
    // A whole sub-block into raw[].  `base`: the matrix plus the sub-block's step.
    __device__ __forceinline__ void load_whole(const char *base, Raw (&raw)[CH]) const
    {
        const GLB_AS char *b = (const GLB_AS char *)uniform_ptr((const uint16_t *)(base + origin));
#pragma unroll
        for (int j = 0; j < CH; ++j)
            raw[j] = load_from(b, rel[j]);
    }
    // Sub-block kb of the tile, which starts at `base`.  tail: the last, incomplete one.
    __device__ __forceinline__ void load_any(const char *base, int64_t kb, bool tail, Raw (&raw)[CH]) const
    {
        base += origin;
        if (TINY && tiny) {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int idx = j * GT + tg;
                if constexpr (KMAJ)
                    raw[j] = gen_gather<KIND>(base + rel[j], K - (kb * SUB + (idx & 7) * E));
                else        // fewer than E columns are the matrix's whole width: column 0 on
                    raw[j] = gen_gather<KIND>(base + rel[j], kb * SUB + idx / Img::CPR < K && idx % Img::CPR == 0 ? run : 0);
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int idx = j * GT + tg;
            int64_t back = 0;
            if constexpr (KMAJ) {
                const int64_t pos = kb * SUB + (idx & 7) * E;
                back = (pos > K - E ? pos - (K - E) : 0) * S;           // the run's last chunk
            } else {
                const int64_t k = kb * SUB + idx / Img::CPR;
                back = (k < K ? 0 : k - (K - 1)) * ld * S;              // the last k-row
            }
            raw[j] = gen_load<KIND>(base + ((int64_t)rel[j] - (tail ? back : 0)));
        }
    }
    __device__ __forceinline__ void finish_whole(LDS_AS char *img, const Raw (&raw)[CH]) const
    {
#pragma unroll
        for (int j = 0; j < CH; ++j)
            *(LDS_AS gu32x4 *)(img + Img::dst_byte(j * GT + tg)) = gen_to_lds<KIND>(raw[j]);
    }
    // With what load_any moved back shifted out and zeros in its place.
    __device__ __forceinline__ void finish_any(LDS_AS char *img, bool tail, const Raw (&raw)[CH]) const
    {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int idx = j * GT + tg;
            Raw v = raw[j];
            if (!(TINY && tiny)) {
                int64_t over;
                if constexpr (KMAJ) {
                    over = tail ? (K - 1) / SUB * SUB + (idx & 7) * E - (K - E) : 0;
                } else {
                    over = first + (int64_t)(idx % Img::CPR) * E - (limit - E);
                    if (tail && (K - 1) / SUB * SUB + idx / Img::CPR >= K)
                        over = E;
                }
                v = gen_shift<KIND>(v, over <= 0 ? 0 : over < E ? (int)over : E);
            }
            *(LDS_AS gu32x4 *)(img + Img::dst_byte(idx)) = gen_to_lds<KIND>(v);
        }
    }
};

template <int KIND, bool A_KMAJ, bool B_KMAJ, int BM, int BN, int WGM, int WGN, int KW>
struct GenConfig {
    static constexpr int GW = WGM * WGN;                    // wavefronts per group
    static constexpr int NT = GW * KW * 64;
    static constexpr uint32_t SUBB = (BM + BN) * 128;       // LDS bytes of one group's sub-block
    static constexpr int EPI_LD = BN + 4;
    static constexpr size_t kLds = 2 * (size_t)KW * SUBB > (size_t)KW * BM * EPI_LD * 4 ? 2 * (size_t)KW * SUBB
                                                                                      : (size_t)KW * BM * EPI_LD * 4;
};

// The end of a tile: KW staged tiles of fp32 (int32) sums in LDS, added in group order, through
// the epilogue to C, or to this slice's partial sums, by all NT threads along the rows.
// HIDE: keep what the addresses are computed from out of the loop before.
template <int KIND, int BM, int BN, int NT, int KW, bool HIDE>
__device__ __forceinline__ void gen_store_sums(const GenArgs &p, LDS_AS char *smem, int tid, int64_t m0, int64_t n0, int slice)
{
    constexpr int EPI_LD = BN + 4;
    int et = tid;
    if constexpr (HIDE)                             // nothing that is computed from it can move into the loop,
        asm volatile("" : "+v"(et));                // where this tile has no register left for it
    LDS_AS float *sums = (LDS_AS float *)smem;
    const bool to_partial = p.split > 1;
    float *part = to_partial ? p.partial + (int64_t)slice * p.M * p.N : nullptr;
    const bool vec = to_partial ? ((p.N & 3) == 0) : ((p.epi.ldc & 3) == 0 && (((uintptr_t)p.epi.C) & 15) == 0);
    auto add = [](float x, float y) {
        if constexpr (KIND == KIND_S8)
            return __int_as_float((int)((uint32_t)__float_as_int(x) + (uint32_t)__float_as_int(y)));
        else
            return x + y;
    };
    constexpr int Q_IT = BM * BN / 4 / NT;
    static_assert(NT % (BN / 4) == 0, "a thread stores the same columns of every row it takes");
    f32x4 old[Q_IT > 0 ? Q_IT : 1], bias = {0.0f, 0.0f, 0.0f, 0.0f};
    const bool accumulate = Q_IT > 0 && accumulates_f32(p.epi, to_partial) && n0 + BN <= p.N;
    if (accumulate) {
        bias = bias4(p.epi, n0 + (et % (BN / 4)) * 4);
#pragma unroll
        for (int i = 0; i < Q_IT; ++i) {
            const int idx = i * NT + et;
            const int64_t m = m0 + idx / (BN / 4);
            old[i] = *(const f32x4 *)((const float *)p.epi.C + (m < p.M ? m : p.M - 1) * p.epi.ldc + n0 + (idx % (BN / 4)) * 4);
        }
    }
    auto summed = [&](int row, int c4) {
        f32x4 v = *(LDS_AS f32x4 *)(sums + row * EPI_LD + c4 * 4);
#pragma unroll
        for (int g = 1; g < KW; ++g) {
            const f32x4 o = *(LDS_AS f32x4 *)(sums + (g * BM + row) * EPI_LD + c4 * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = add(v[e], o[e]);
        }
        return v;
    };
    if (accumulate) {
#pragma unroll
        for (int i = 0; i < Q_IT; ++i) {
            const int idx = i * NT + et;
            const int row = idx / (BN / 4), c4 = idx % (BN / 4);
            if (m0 + row < p.M)
                store4_accumulated(p.epi, m0 + row, n0 + c4 * 4, old[i], bias, summed(row, c4));
        }
    } else if (vec) {
#pragma unroll 2
        for (int idx = et; idx < BM * BN / 4; idx += NT) {
            const int row = idx / (BN / 4), c4 = idx % (BN / 4);
            const f32x4 v = summed(row, c4);
            const int64_t m = m0 + row, n = n0 + c4 * 4;
            if (m < p.M) {
                if (to_partial)
                    store4_partial(part + m * p.N + n, p.N - n, true, v[0], v[1], v[2], v[3]);
                else
                    store4_epilogue(p.epi, m, n, p.N - n, true, v[0], v[1], v[2], v[3]);
            }
        }
    } else if constexpr (Q_IT == 0) {
        // (fewer groups of four than threads: one element per thread shares the sums better.
        // 1 x 11 x 626, NN bf16, 32 x 32 tile: 6.0 us, in groups of four 6.7)
        for (int idx = et; idx < BM * BN; idx += NT) {
            const int row = idx / BN, col = idx % BN;
            float v = sums[row * EPI_LD + col];
#pragma unroll
            for (int g = 1; g < KW; ++g)
                v = add(v, sums[(g * BM + row) * EPI_LD + col]);
            const int64_t m = m0 + row, n = n0 + col;
            if (m < p.M && n < p.N) {
                if (to_partial)
                    part[m * p.N + n] = v;
                else
                    epilogue_store(p.epi, v, m, n);
            }
        }
    } else {
#pragma unroll 2
        for (int idx = et; idx < BM * BN / 4; idx += NT) {
            const int row = idx / (BN / 4), c4 = idx % (BN / 4);
            const f32x4 v = summed(row, c4);
            const int64_t m = m0 + row, n = n0 + c4 * 4;
            if (m < p.M) {
                if (!to_partial) {
                    gen_store4(p.epi, m, n, p.N - n, v);
                } else if (n + 4 <= p.N) {
                    *(f32x4_any4 *)(part + m * p.N + n) = v;
                } else {
                    store4_partial(part + m * p.N + n, p.N - n, false, v[0], v[1], v[2], v[3]);
                }
            }
        }
    }
}

// ROWS_SHORT: an operand's contiguous run is shorter than a chunk (K or an m/n extent of a few
// elements), so its chunks are gathered element by element; a kernel of its own, because
// that path's varying number of loads would make every wait of the loop a full one.  ROWS_FAR: rows so far apart
// that a tile's offsets do not fit 32 bits.
template <int KIND, bool A_KMAJ, bool B_KMAJ, int BM, int BN, int WGM, int WGN, int KW, bool HAS_OFF, int ROWS>
__global__ void __launch_bounds__(WGM *WGN *KW * 64, WGM *WGN > 1 ? 4 : 2)
general_kernel(GenArgs p)
{
    typedef GenConfig<KIND, A_KMAJ, B_KMAJ, BM, BN, WGM, WGN, KW> Cfg;
    constexpr int GW = Cfg::GW, GT = GW * 64, NT = Cfg::NT;
    constexpr int CA = BM * 8 / GT, CB = BN * 8 / GT;       // chunks per thread and operand
    static_assert(CA * GT == BM * 8 && CB * GT == BN * 8, "whole chunks per thread");
    constexpr bool F32 = KIND == KIND_F32;
    constexpr int MT = F32 ? 32 : 16;                       // matrix instruction tile
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / MT, TN = WN / MT;
    typedef GenLoader<KIND, BM, A_KMAJ, CA, GT, ROWS> LoadA;
    typedef GenLoader<KIND, BN, B_KMAJ, CB, GT, ROWS> LoadB;
    typedef typename LoadA::Img ImgA;
    typedef typename LoadB::Img ImgB;
    constexpr int S = GenElem<KIND>::S, SUB = GenElem<KIND>::SUB;

    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    LDS_AS char *smem = (LDS_AS char *)smem_generic;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = w / GW, wg = w % GW;                     // k group, wave in the group
    const int wm = wg / WGN, wn = wg % WGN;
    const int tg = wg * 64 + lane;

    const int64_t z = blockIdx.z;
    const char *Abase = p.A + z * p.ms_a * S, *Bbase = p.B + z * p.ms_b * S;
    p.epi.C = (char *)p.epi.C + z * p.ms_c * (p.epi.c_f32 ? 4 : 2);

    int tile, slice, tm, tn;
    slice_major_coords(p.tiles_m * p.tiles_n, p.split, p.walk, tile, slice);
    group_walk(tile, p.tiles_m, p.tiles_n, p.walk, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    // Reduction range of this workgroup: flattened (batch, sub-block) steps, dealt to the
    // groups in turn: group kg takes steps begin + kg, begin + kg + KW, ...
    const int64_t kbs = (p.K + SUB - 1) / SUB;
    const int64_t total = p.batch * kbs;
    const int64_t per = p.walk.per;
    const int64_t begin = slice * per < total ? slice * per : total;
    const int64_t end = begin + per < total ? begin + per : total;
    const int64_t rounds = (end - begin + KW - 1) / KW;
    const bool k_ragged = p.K % SUB != 0;

    LoadA la;
    LoadB lb;
    la.init(tg, m0, p.M, p.lda, p.K, false);
    lb.init(tg, n0, p.N, p.ldb, p.K, p.b_packed != 0);

    f32x4 acc16[F32 ? 1 : TN][F32 ? 1 : TM];
    f32x16 acc32[F32 ? TN : 1][F32 ? TM : 1];
    if constexpr (F32) {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc32[a][b][r] = 0.0f;
    } else {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc16[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    auto multiply = [&](int stage) {
        LDS_AS char *at = smem + (uint32_t)(stage * KW + kg) * Cfg::SUBB;
        LDS_AS char *bt = at + ImgA::BYTES;
        if constexpr (F32) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 fa[TM], fb[TN];
#pragma unroll
                for (int t = 0; t < TM; ++t)
                    fa[t] = ImgA::frag32(at, wm * WM, t, j, lane);
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    fb[t] = ImgB::frag32(bt, wn * WN, t, j, lane);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int a = 0; a < TN; ++a)
#pragma unroll
                        for (int b = 0; b < TM; ++b)
                            acc32[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[a][e], fa[b][e], acc32[a][b], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                bf16x8 fa[TM], fb[TN];
#pragma unroll
                for (int t = 0; t < TM; ++t)
                    fa[t] = ImgA::frag16(at, wm * WM, t, st, lane);
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    fb[t] = ImgB::frag16(bt, wn * WN, t, st, lane);
#pragma unroll
                for (int a = 0; a < TN; ++a)
#pragma unroll
                    for (int b = 0; b < TM; ++b)
                        acc16[a][b] = mfma_16x16x32<kind_is_f8(KIND) ? KIND_BF16 : KIND>(fb[a], fa[b], acc16[a][b]);
            }
        }
    };
    // A group of one wavefront owns its LDS alone: its own waits order everything, and the
    // groups run free of one another.  Larger groups share a stage and meet once per step.
    auto meet = [&]() {
        wait_lgkmcnt0();
        if constexpr (GW > 1)
            block_sync();
        else
            asm volatile("" ::: "memory");
    };

    // The loop, in two forms.  Whole sub-blocks at whole tiles (EDGES = false) need no shift
    // and no branch: the K tail is then taken FIRST (step 0 stands for the last sub-block,
    // step u for sub-block u - 1), outside the loop.  Tiles that overhang an m/n-contiguous
    // operand, and a batch-reduce with a K tail in every tile, shift every chunk.
    // The cursor of a group stops at the last step of all, whose loads are then repeated
    // (and never multiplied).
    struct Set {
        typename LoadA::Raw a[CA];
        typename LoadB::Raw b[CB];
        bool tail;
    };
    auto run = [&](auto edges) {
        constexpr bool EDGES = decltype(edges)::value;
        const int64_t rot = !EDGES && k_ragged ? 1 : 0;
        int64_t u = begin + kg < total ? begin + kg : total - 1;
        int64_t i = 0, kb = u - rot;
        TileOffsets offs_a, offs_b;
        if constexpr (HAS_OFF) {
            i = p.walk.by_kblocks.mul ? div_by((int)u, p.walk.by_kblocks) : u / kbs;
            kb = u - i * kbs;
            offs_a.init(p.A_off, p.batch, (int)i, lane);
            offs_b.init(p.B_off, p.batch, (int)i, lane);
        }
        // Step 0 of this group is the tail (any other sub-block is whole, and needs none of what the tail does).
        const bool tail0 = rot && kb < 0;
        auto issue = [&](Set &s, auto first) {
            const char *a = Abase, *b = Bbase;
            if constexpr (HAS_OFF) {
                a += offs_a.get((int)i, lane) * S;
                b += offs_b.get((int)i, lane) * S;
            }
            if (EDGES || (decltype(first)::value && tail0)) {
                const int64_t at = kb < 0 ? kbs - 1 : kb;
                s.tail = k_ragged && at == kbs - 1;
                la.load_any(a + at * la.step, at, s.tail, s.a);
                lb.load_any(b + at * lb.step, at, s.tail && !lb.packed, s.b);
            } else {
                // (a cursor that stays on the tail's step repeats sub-block 0, which is whole)
                const int64_t at = kb < 0 ? 0 : kb;
                la.load_whole(a + at * la.step, s.a);
                lb.load_whole(b + at * lb.step, s.b);
            }
            if (u + KW < total) {
                u += KW;
                kb += KW;
                if constexpr (HAS_OFF) {
                    while (kb >= kbs) {
                        kb -= kbs;
                        ++i;
                    }
                }
            }
        };
        auto finish = [&](const Set &s, int stage, auto first) {
            LDS_AS char *at = smem + (uint32_t)(stage * KW + kg) * Cfg::SUBB;
            if (EDGES || (decltype(first)::value && tail0)) {
                la.finish_any(at, s.tail, s.a);
                lb.finish_any(at + ImgA::BYTES, s.tail && !lb.packed, s.b);
            } else {
                la.finish_whole(at, s.a);
                lb.finish_whole(at + ImgA::BYTES, s.b);
            }
        };
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        Set set0;
        issue(set0, yes);
        if constexpr (BM == 128) {
            // Two sets of registers in turn, each requested two steps ahead.  Every step
            // requests (the last ones repeat, see the cursor), and steps come in pairs (one
            // past the end multiplies nothing): with a number of loads that differs from
            // path to path the compiler would wait for the younger set as well.
            Set set1;
            auto step = [&](int64_t t, Set &s, auto stage) {
                constexpr int cur = decltype(stage)::value;
                finish(s, cur ^ 1, no);                 // step t + 1
                issue(s, no);                           // step t + 3
                if (begin + kg + t * KW < end)
                    multiply(cur);
                meet();                                 // step t read, step t + 1 written
            };
            issue(set1, no);
            finish(set0, 0, yes);
            issue(set0, no);
            meet();
            for (int64_t t = 0; t < rounds; t += 2) {
                step(t, set1, std::integral_constant<int, 0>{});
                step(t + 1, set0, std::integral_constant<int, 1>{});
            }
        } else {
            // One set, one step ahead: these tiles are for few steps, where the surplus
            // requests of the deeper form cost more than it hides.
            finish(set0, 0, yes);
            if (rounds > 1)
                issue(set0, no);
            meet();
            for (int64_t t = 0; t < rounds; ++t) {
                const int cur = (int)(t & 1);
                if (t + 1 < rounds)
                    finish(set0, cur ^ 1, no);
                if (t + 2 < rounds)
                    issue(set0, no);
                if (begin + kg + t * KW < end)
                    multiply(cur);
                meet();
            }
        }
    };
    // (A single, incomplete sub-block has no whole one to repeat.)
    if (la.edge || lb.edge || ROWS == ROWS_SHORT || (k_ragged && (HAS_OFF || kbs == 1)))
        run(std::true_type{});
    else
        run(std::false_type{});
    if constexpr (GW == 1)
        block_sync();                               // the staging below reuses every group's LDS

    // ---- epilogue through LDS: every group's tile row-wise, added in group order, stored
    // by all threads along the rows, four elements per lane whatever C's alignment (32 x 32 tiles: one).  (One element
    // per lane where rows are not 16-byte aligned bounds a short reduction: 4001 x 4003 x 31, 128 x 128
    // tiles, bf16 37.5 -> 30.5 us, fp32 35.8 -> 29.5, int8 31.5 -> 27.6; 2001 x 2003 x 31 15.8 -> 14.4.)
    LDS_AS float *stage = (LDS_AS float *)smem + (size_t)kg * BM * Cfg::EPI_LD;
    if constexpr (F32) {
        static_for<0, TN * TM>([&](auto ic) {
            constexpr int a = decltype(ic)::value / TM, b = decltype(ic)::value % TM;
            static_for<0, 4>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                *(LDS_AS f32x4 *)(stage + (wm * WM + 32 * b + (lane & 31)) * Cfg::EPI_LD + wn * WN + 32 * a + 8 * q + 4 * (lane >> 5)) =
                    f32x4{acc32[a][b][4 * q], acc32[a][b][4 * q + 1], acc32[a][b][4 * q + 2], acc32[a][b][4 * q + 3]};
            });
        });
    } else {
        static_for<0, TN * TM>([&](auto ic) {
            constexpr int a = decltype(ic)::value / TM, b = decltype(ic)::value % TM;
            *(LDS_AS f32x4 *)(stage + (wm * WM + 16 * b + (lane & 15)) * Cfg::EPI_LD + wn * WN + 16 * a + 4 * (lane >> 4)) =
                acc16[a][b];
        });
    }
    wait_lgkmcnt0();
    block_sync();
    gen_store_sums<KIND, BM, BN, NT, KW, BM * BN == 128 * 128>(p, smem, tid, m0, n0, slice);
}

inline GenArgs gen_args(const Problem &p)
{
    GenArgs a;
    a.M = p.M; a.N = p.N; a.K = p.K; a.batch = p.batch;
    a.A = (const char *)p.A; a.A_off = p.A_off; a.lda = p.lda;
    a.B = (const char *)p.B; a.B_off = p.B_off; a.ldb = p.ldb;
    a.b_packed = p.b_packed;
    a.epi.beta = p.beta; a.epi.C = p.C; a.epi.ldc = p.ldc; a.epi.c_f32 = p.c_f32; a.epi.c_f16 = p.in_f16;
    a.epi.c_i32 = p.in_s8; a.epi.bias = p.bias; a.epi.relu = p.relu;
    a.split = p.split; a.partial = p.partial;
    a.ms_a = p.ms_a; a.ms_b = p.ms_b; a.ms_c = p.ms_c;
    return a;
}

template <int KIND, bool A_KMAJ, bool B_KMAJ, int BM, int BN, int WGM, int WGN, int KW, bool HAS_OFF, int ROWS = ROWS_NEAR>
hipError_t general_launch(const Problem &p)
{
    typedef GenConfig<KIND, A_KMAJ, B_KMAJ, BM, BN, WGM, WGN, KW> Cfg;
    GenArgs a = gen_args(p);
    const int64_t tm = (p.M + BM - 1) / BM, tn = (p.N + BN - 1) / BN;
    if (tm * tn * Cfg::NT > 0xffffffffLL)           // (the host cuts such problems first)
        return hipErrorInvalidValue;
    a.tiles_m = (int)tm;
    a.tiles_n = (int)tn;
    a.walk = make_walk(a.tiles_m, a.tiles_n, p.split, (p.K + GenElem<KIND>::SUB - 1) / GenElem<KIND>::SUB, p.batch, (int64_t)kWalkRows * tn);
    const dim3 grid((unsigned)(tm * tn), (unsigned)p.split, (unsigned)p.nmat);
    void (*kern)(GenArgs) = general_kernel<KIND, A_KMAJ, B_KMAJ, BM, BN, WGM, WGN, KW, HAS_OFF, ROWS>;
    static thread_local bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Cfg::kLds);
        if (e != hipSuccess)
            return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(Cfg::NT), Cfg::kLds, p.stream, a);
    return hipGetLastError();
}

}  // namespace brg

#include "general_duty.hpp"

namespace brg {

// The undivided kernel's tiles.
template <int KIND, bool A_KMAJ, bool B_KMAJ, bool HAS_OFF, int ROWS>
hipError_t general_undivided(const Problem &p, int tile)
{
    switch (tile) {
    case GEN_128: return general_launch<KIND, A_KMAJ, B_KMAJ, 128, 128, 2, 4, 1, HAS_OFF, ROWS>(p);
    case GEN_MID: return general_launch<KIND, A_KMAJ, B_KMAJ, 128, 64, 4, 2, 1, HAS_OFF, ROWS>(p);
    case GEN_64: return general_launch<KIND, A_KMAJ, B_KMAJ, 64, 64, 2, 2, 2, HAS_OFF, ROWS>(p);
    default: return general_launch<KIND, A_KMAJ, B_KMAJ, 32, 32, 1, 1, 8, HAS_OFF, ROWS>(p);
    }
}

// ROWS_FAR: general_launch_far's instances (neither divided nor tuned kernels take such rows); else all others.
template <int KIND, bool A_KMAJ, bool B_KMAJ, bool HAS_OFF, int ROWS>
hipError_t general_tile(const Problem &p, int tile)
{
    if constexpr (ROWS == ROWS_FAR) {
        return general_undivided<KIND, A_KMAJ, B_KMAJ, HAS_OFF, ROWS>(p, tile);
    } else {
        if (general_short_runs(p))
            return general_launch<KIND, A_KMAJ, B_KMAJ, 64, 64, 2, 2, 2, HAS_OFF, ROWS_SHORT>(p);
        if constexpr (!HAS_OFF) {
            if constexpr (KIND == KIND_BF16 || KIND == KIND_F16) {
                if (tile == GEN_128 && tail_kernel(p, p.split) != TAIL_NONE)
                    return launch_tail(p);
                if (tile == GEN_128 && realign_wins(p))
                    return launch_realigned(p);
                if (stream_form_runs(p, tile))
                    return launch_stream_form(p, tile);
            }
            if (duty_runs(p, tile))
                return duty_tile<KIND, A_KMAJ, B_KMAJ>(p, tile);
        }
        return general_undivided<KIND, A_KMAJ, B_KMAJ, HAS_OFF, ROWS_NEAR>(p, tile);
    }
}

template <int KIND, bool HAS_OFF, int ROWS = ROWS_NEAR>
hipError_t general_layout(const Problem &p, int tile)
{
    const bool ak = p.transA == 0, bk = p.transB == 1 || p.b_packed;
    if (ak)
        return bk ? general_tile<KIND, true, true, HAS_OFF, ROWS>(p, tile) : general_tile<KIND, true, false, HAS_OFF, ROWS>(p, tile);
    return bk ? general_tile<KIND, false, true, HAS_OFF, ROWS>(p, tile) : general_tile<KIND, false, false, HAS_OFF, ROWS>(p, tile);
}

}  // namespace brg
