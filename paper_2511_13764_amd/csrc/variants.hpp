// Kernel variants and the host-side plan (which variant, how many reduction
// splits).  Tile selection is by hand-tuned rule, as in Section 5(a) of the
// paper (tile sizes are chosen per target by sweeping).
#pragma once
#include "common.hpp"

namespace brg {

enum Variant {
    V_GENERIC = 0,      // any shape / alignment (general.hpp, general_short.hip), its tile by size
    V_BF16_128x128,     // bf16, 128x128x64 workgroup tile, 64x64 wave tile
    V_BF16_PP256,       // bf16, 256x256x64 tile, 8 waves in alternating memory/compute phases
    V_F32_128x128,      // fp32, 128x128x32 tile, fp32 MFMA
    V_BF16_STREAM32,    // bf16, skinny M: 32x128x64 tile, deep LDS ring (HBM-bound shapes)
    V_BF16_STREAM64,    // bf16, skinny M: 64x128x64 tile, deep LDS ring
    V_BF16_STREAM128,   // bf16, skinny M: 128x128x64 tile, deep LDS ring
    V_COUNT
};

constexpr int kMaxSplit = 16;
constexpr int64_t kMaxShort = 32;       // longest reduction of the general path's short kernel

// Tiles of the general kernel.  As waves that load beside waves that multiply (duty_runs): 128 x 128 and 128 x 64 (4 or 8 + 4
// waves), 64 x 64 (4 + 4).  Undivided: 128 x 128 and 128 x 64 (8 waves), 64 x 64 (2 groups of 4 waves share the reduction), 32 x 32
// (8 groups of one wave; always).  GEN_128 also stands for the tuned kernels behind it (tail_kernel, realign_wins).
enum GenTile { GEN_128, GEN_MID, GEN_64, GEN_32, GEN_TILES,
               FORM_NARROW = GEN_TILES,         // 48-column form of the 128-row streaming kernel
               FORM_SHORT };                    // general path, short reductions: general_short.hip

struct Plan {
    int variant;
    int split;          // of the launch itself: 1 writes no partial tiles and needs no workspace
    int form;           // tile of the general kernel (GenTile); -1: the variant's own kernel.  Where
                        // full tiles leave CUs idle a tuned variant has a reduced-tile form: the general
                        // kernel's 64- or 32-wide tiles, 128 x 64 (stream_form_runs), or FORM_NARROW; none is split
    int displaced = 0;  // split of the plan that split_for_streamed_b took the place of, or 0
};

const char *variant_name(int v);
const char *form_name(int form);

// Pick variant, split and form for a validated, non-empty problem.  forced_variant < 0,
// forced_split <= 0 and forced_form < 0 mean automatic.  Returns a BRGEMM_* code.
int choose_plan(const Problem &p, size_t workspace_bytes, int forced_variant, int forced_split, int forced_form, Plan *out);

// True when a contiguous run of an operand (K, or the m/n extent of an m/n-contiguous operand)
// is shorter than a 16-byte chunk (FP8: 8 values): the general kernel then gathers its chunks.
inline bool general_short_runs(const Problem &p)
{
    const int64_t chunk = in_16bit(p) || p.in_f8 ? 8 : p.in_s8 ? 16 : 4;
    return (p.transA ? p.M : p.K) < chunk || (!p.b_packed && (p.transB ? p.K : p.N) < chunk);
}

// True when a chunk's place in an operand's part of a tile fits the 32 bits that the general kernel keeps it in: (rows - 1) * pitch
// and the place along the row.  Rows of a tile are the matrix's rows that it spans; of an m/n-contiguous operand a sub-block's
// k-rows (those past the last are formed, too, before they are moved back); of packed B eight groups of k.  The
// others run in the same tiles with 64 bits (general_far.hip).
inline bool general_offsets_fit(const Problem &p, int tile)
{
    const int64_t s = in_16bit(p) ? 2 : in_8bit(p) ? 1 : 4, sub = p.in_s8 ? 128 : s == 4 ? 32 : 64;
    const int64_t bm = tile == GEN_32 ? 32 : tile == GEN_64 ? 64 : 128, bn = tile == GEN_128 ? 128 : tile == GEN_32 ? 32 : 64;
    const int64_t rows_a = p.transA ? sub : p.M < bm ? p.M : bm;
    const int64_t rows_b = p.b_packed ? 8 : p.transB == 0 ? sub : p.N < bn ? p.N : bn;
    const int64_t most = (((int64_t)1 << 32) - 4096) / s;       // (along a row: at most 128 columns of 8 packed values)
    return (rows_a == 1 || p.lda <= most / (rows_a - 1)) && (rows_b == 1 || p.ldb <= most / (rows_b - 1));
}

// True when the general kernel's wide tiles can run as loading and multiplying waves
// (general_duty.hpp): one product of at least four sub-blocks of k, whose tiles are addressed in 32 bits.
inline bool duty_eligible(const Problem &p)
{
    const int64_t s = in_16bit(p) ? 2 : in_8bit(p) ? 1 : 4, sub = p.in_s8 ? 128 : s == 4 ? 32 : 64;
    const int64_t steps = (p.K + sub - 1) / sub;
    return p.batch == 1 && !p.A_off && p.lda * s < (1 << 23) && p.ldb * s < (1 << 23) && steps >= 4 &&
           steps < ((int64_t)1 << 30) && !general_short_runs(p);
}

// An automatic plan of a small grid: other tiles where they are faster than the tuned kernel of the table.
void prefer_small_tiles(const Problem &p, size_t workspace_bytes, Plan *io);

// True when `v` can run `p` (alignment and layout rules of the tuned kernels).
bool variant_eligible(int v, const Problem &p);

hipError_t launch_variant(int v, const Problem &p);

// general_half.hip, general_bytes.hip, general_f32.hip, general_offsets.hip: one translation
// unit per class of operands, which build side by side
hipError_t general_launch_half(const Problem &p, int tile);
hipError_t general_launch_bytes(const Problem &p, int tile);
hipError_t general_launch_f32(const Problem &p, int tile);
hipError_t general_launch_offsets(const Problem &p, int tile);
hipError_t general_launch_short(const Problem &p);
hipError_t general_launch_far(const Problem &p, int tile);          // general_far.hip, general_far_offsets.hip
hipError_t general_launch_far_offsets(const Problem &p, int tile);
// bf16_mfma.hip
bool bf16_mfma_eligible(const Problem &p);
bool bf16_rows_eligible(const Problem &p);
hipError_t launch_bf16_128x128(const Problem &p);
// bf16_wide.hip: the 128 x 256 tile that the variant launches on an unsplit problem where it is faster
bool wide_tile_wins(const Problem &p);
hipError_t launch_bf16_wide(const Problem &p);
// f32_mfma.hip
bool f32_mfma_eligible(const Problem &p);
hipError_t launch_f32_128x128(const Problem &p);
// bf16_pingpong.hip
bool bf16_pingpong_eligible(const Problem &p);
hipError_t launch_bf16_pingpong(const Problem &p);

// pingpong_tail.hip
hipError_t launch_pingpong_tail(const Problem &p);

// General path, 128 x 128 form: the kernel of a tuned variant that takes the problem although K is no
// multiple of 64 (its incomplete block goes through registers).
enum TailKernel { TAIL_NONE, TAIL_NARROW, TAIL_128, TAIL_WIDE, TAIL_PINGPONG };
TailKernel tail_kernel(const Problem &p, int split);
hipError_t launch_tail(const Problem &p);
hipError_t launch_stream_tail(const Problem &p, TailKernel k);      // stream_tail.hip

// realign.hip: the same form for rows that the tuned kernels cannot read, copied into the workspace first
bool realign_wins(const Problem &p);
hipError_t launch_realigned(const Problem &p);
bool realign_pays(const Problem &p, size_t bytes);      // dispatch.hip

// bf16_stream.hip
bool bf16_stream_eligible(const Problem &p, int bm);
int stream_tile_instead(const Problem &p, int bm, int split);      // a GenTile, or -1: its full tiles
hipError_t launch_bf16_stream(const Problem &p, int bm);
hipError_t launch_bf16_stream_narrow(const Problem &p);

// bf16_stream64.hip: the general path's 64 x 64 and 128 x 64 forms on 16-bit rows that global->LDS loads can read
bool stream_form_runs(const Problem &p, int tile);
hipError_t launch_stream_form(const Problem &p, int tile);

}  // namespace brg
