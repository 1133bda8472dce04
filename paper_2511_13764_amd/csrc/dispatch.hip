// Variant table, eligibility rules and the automatic plan.
#include "../../include/brgemm.h"
#include "variants.hpp"

namespace brg {

const char *variant_name(int v)
{
    switch (v) {
    case V_GENERIC: return "generic_64x64x16_f32mfma";      // the first general kernel's name, which programs compare; its tile is its form
    case V_BF16_128x128: return "bf16_128x128x64";
    case V_BF16_PP256: return "bf16_pingpong_256x256x64";
    case V_F32_128x128: return "f32_128x128x32";
    case V_BF16_STREAM32: return "bf16_stream_32x128x64";
    case V_BF16_STREAM64: return "bf16_stream_64x128x64";
    case V_BF16_STREAM128: return "bf16_stream_128x128x64";
    default: return "";
    }
}

const char *form_name(int form)
{
    switch (form) {
    case GEN_128: return "128x128";
    case GEN_MID: return "128x64";
    case GEN_64: return "64x64";
    case GEN_32: return "32x32";
    case FORM_NARROW: return "128x48";
    case FORM_SHORT: return "64x64 short";
    default: return "";
    }
}

// Which tuned variants have which form (V_GENERIC has the four tiles of the general kernel and the
// kernel for short reductions).  FP8 has no reduced tiles: the general kernel multiplies it as bf16,
// so the rounding of a sum would depend on the size of the grid; their time was not measured.
static bool form_eligible(int form, int variant, const Problem &p)
{
    if (form == FORM_NARROW)
        return variant == V_BF16_STREAM128 && in_16bit(p) && p.transA == 0 && p.transB == 1 && !p.A_off;
    if (form == FORM_SHORT)
        return variant == V_GENERIC && p.batch == 1 && p.K <= kMaxShort;
    if (variant == V_GENERIC)
        return form < GEN_TILES && (form == GEN_64 || !general_short_runs(p));
    if (form == GEN_MID)
        return (variant == V_BF16_STREAM32 || variant == V_BF16_STREAM64) && stream_form_runs(p, form);
    return (form == GEN_64 || form == GEN_32) && !p.in_f8 && variant != V_BF16_PP256 && variant != V_BF16_128x128;
}

bool variant_eligible(int v, const Problem &p)
{
    switch (v) {
    case V_GENERIC: return true;
    case V_BF16_128x128: return bf16_mfma_eligible(p) && !p.in_f8;      // no 32x32 FP8 form here
    case V_BF16_PP256: return bf16_pingpong_eligible(p);
    case V_F32_128x128: return f32_mfma_eligible(p);
    case V_BF16_STREAM32: return bf16_stream_eligible(p, 32);
    case V_BF16_STREAM64: return bf16_stream_eligible(p, 64);
    case V_BF16_STREAM128: return bf16_stream_eligible(p, 128);
    default: return false;
    }
}

static size_t split_bytes(const Problem &p, int split)
{
    return split > 1 ? (size_t)split * (size_t)p.M * (size_t)p.N * sizeof(float) : 0;
}

// Reduction split for a grid of 128x128 tiles that cannot fill the chip (skinny M,
// small squares, batch-reduce into a small C).  A rough time model, in microseconds,
// with constants fitted to split sweeps on MI355X: a 128x128x64 k-block costs ~0.57 us
// per workgroup, 512 workgroups run at once (two per CU), streaming the operands cannot
// beat ~8 TB/s (they sit in the Infinity Cache when a call repeats), and the fixed-order reduction moves split*M*N*8 bytes at ~3 TB/s plus
// a second launch.
static int split_for_small_grid(const Problem &p, size_t workspace_bytes)
{
    const double tiles = (double)((p.M + 127) / 128) * (double)((p.N + 127) / 128);
    const double kblocks = (double)p.batch * (double)(p.K / 64);
    const double operand_bytes = 2.0 * ((double)p.M + (double)p.N) * (double)p.K * (double)p.batch;
    static const int candidates[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    int best = 1;
    double best_t = 1e30;
    for (int s : candidates) {
        if (s > kMaxSplit || (s > 1 && kblocks / s < 2.0))
            continue;
        if (s > 1 && (size_t)s * (size_t)p.M * (size_t)p.N * sizeof(float) > workspace_bytes)
            continue;
        const double rounds = (double)(int64_t)((tiles * s + 511.0) / 512.0);
        double t_main = rounds * (kblocks / s) * 0.57;
        const double t_stream = operand_bytes / 8.0e6;
        if (t_main < t_stream)
            t_main = t_stream;
        const double t_reduce = s > 1 ? 4.0 + (double)s * (double)p.M * (double)p.N * 8.0 / 3.0e6 : 0.0;
        const double t = 6.0 + t_main + t_reduce;
        if (t < best_t * 0.97) {     // prefer the smaller split on near ties
            best_t = t;
            best = s;
        }
    }
    return best;
}

// Reduction split for the skinny-M streaming kernels (BM x 128 tiles).  Split sweeps
// on the MLP shapes show the time following rounds * (k-blocks per workgroup), where
// rounds = workgroups / 256 rounded up (a CU works through its workgroups at a fixed
// rate), plus a cost per split for the partial tiles that grows with BM.
static int split_for_stream(const Problem &p, int bm, size_t workspace_bytes)
{
    const int64_t tiles = ((p.M + bm - 1) / bm) * ((p.N + 127) / 128);
    const int64_t kblocks = p.batch * (p.K / 64);
    const double per_split = 0.75 * bm / 32.0;
    int best = 1;
    double best_cost = 1e30;
    for (int s = 1; s <= kMaxSplit; ++s) {
        const int64_t per = (kblocks + s - 1) / s;
        if (s > 1 && (per < 8 || split_bytes(p, s) > workspace_bytes))
            continue;
        const double rounds = (double)((tiles * s + 255) / 256);
        const double cost = rounds * (double)per + per_split * s;
        if (cost < best_cost) {
            best_cost = cost;
            best = s;
        }
    }
    return best;
}

// Tile height and reduction split for a grid of at most 256 tiles of 128 x 128 (small
// squares, batch-reduce into a small C): operands that sit in L2 / the Infinity Cache, so
// what counts is how many CUs have work and what a k-block costs a workgroup.  Shorter
// tiles put more workgroups on the chip (1024^3: 256 tiles of 32 x 128 take 9.3 us, 64
// tiles of 128 x 128 take 12.4), as long as they still all run at once; two workgroups of
// the 32- and 64-row kernels share a CU.  Time model in microseconds, constants from
// sweeps over 512^3 ... 2048^3, 512 x 512 x 4096 and the scattered batch-reduce
// configuration: a k-block costs a workgroup 0.20 / 0.29 / 0.42 us at 32 / 64 / 128 rows
// (twice that for a batch-reduce over scattered tiles, where every 64-deep block is a new tile
// somewhere else in memory), a split
// costs a second launch (4.5 us) plus writing and reading its partial tiles.
static void plan_small_grid(const Problem &p, size_t workspace_bytes, bool may_split, int *bm_out, int *split_out)
{
    static const int heights[] = {128, 64, 32};
    static const double block_us[] = {0.42, 0.29, 0.20};
    const int64_t kblocks = p.batch * (p.K / 64);
    double best_t = 1e30;
    *bm_out = 128;
    *split_out = 1;
    // A B operand far larger than the L2s (4 MiB per XCD) is streamed, and every further
    // row of tiles streams it again: then only the tallest tile is considered (measured:
    // 256 x 4096 x 4096 takes 19.0 us as 128-row tiles with split 3 and 24.6 us as 32-row
    // tiles; 1024 x 2048 x 8192 39.8 against 48.9 us with 64-row tiles).
    const bool b_streams = (double)p.N * (double)p.K * (double)p.batch * 2.0 > 8.0 * 1024 * 1024 && p.M > 128;
    for (int i = 0; i < 3; ++i) {
        const int bm = heights[i];
        if (!bf16_stream_eligible(p, bm) || (bm < 128 && p.in_f8))
            continue;
        if (bm < 128 && b_streams && bf16_stream_eligible(p, 128))
            continue;
        const int64_t tiles = ((p.M + bm - 1) / bm) * ((p.N + 127) / 128) * p.nmat;
        if (bm < 128 && tiles > 256)
            continue;
        const int64_t at_once = bm == 128 ? 256 : 512;
        for (int s = 1; s <= (may_split ? kMaxSplit : 1); ++s) {
            const int64_t per = (kblocks + s - 1) / s;
            if (s > 1 && (per < 2 || split_bytes(p, s) > workspace_bytes))
                continue;
            const double rounds = (double)((tiles * s + at_once - 1) / at_once);
            double t = rounds * (double)per * block_us[i] * (p.A_off ? 2.0 : 1.0);
            if (s > 1)
                t += 4.5 + (double)s * (double)p.M * (double)p.N * 4.0 / 4.0e6;
            if (t < best_t * 0.97) {     // near ties: the taller tile, the smaller split
                best_t = t;
                *bm_out = bm;
                *split_out = s;
            }
        }
    }
}

// Split of 256 x 256 tiles that fill the chip, up to `most` slices, where the time model of split_for_mid_grid is below best_t; else 0.
static int pingpong_split(const Problem &p, size_t workspace_bytes, int most, double best_t)
{
    const double kblocks = (double)p.batch * (double)(p.K / 64);
    const int64_t pp_tiles = ((p.M + 255) / 256) * ((p.N + 255) / 256);
    int best = 0;
    for (int s = 2; s <= most; ++s) {
        if (pp_tiles * s > 256 || kblocks / s < 16.0 || split_bytes(p, s) > workspace_bytes)
            continue;
        const double per = (double)(int64_t)((kblocks + s - 1) / s);
        const double mn = (double)p.M * (double)p.N;
        const double t = 12.0 + per * 1.22 + 4.0 + (s * mn * 4.0 + mn * 2.0) / 5.0e6;
        if (t < best_t) {
            best_t = t;
            best = s;
        }
    }
    return best;
}

// Reduction split for the fp32 kernel when its 128x128 tiles cannot fill the chip.
// Time model in microseconds, fitted to split sweeps (256^3 ... 2048^3 and the skinny
// MLP shape): one workgroup per CU works through a 128x128x32 k-block in ~2.0 us
// (the fp32 MFMA rate), a launch costs ~8 us of latency, and the reduction adds a
// second launch plus split*M*N*8 bytes at ~3 TB/s.
// Between 257 and 512 tiles of 128 x 128: either the two-stage 128 x 128 kernel with two
// workgroups per CU (about 1.0 us per k-block when all 512 are there) or the 256 x 256
// kernel on a quarter as many tiles with the reduction split so that they fill the chip
// (1.22 us per k-block, plus the partial tiles: split * M * N * 4 bytes read and the
// result written at ~5 TB/s, plus a second launch).  Measured: 2048 x 4096 x 11008 takes
// 174 us the first way and 144 us the second (split 2), 1024 x 8192 x 8192 131 against
// 113 us; at K = 4096 the two are level.  Or one round of 128 x 256 tiles, 0.65 us per k-block
// with half of the CUs at work, 0.83 with all (the chip's clock): on 75 problems (352 x 10936 ... 4064 x 1120,
// K 3200 to 12160) that it takes from 256 x 256 tiles with split 2 or 3, 0.75 to 1.03 of their time, 0.88 on average.
// Not where the sum stays in fp32: one chain of additions over all of K is further from the exact sum than
// the split's two or three (1049 x 3840 x 6208: 4.9e-7 of the result against 2.8e-7).  Returns the split for the 256 x 256
// kernel, or 0 to stay with the variant bf16_128x128x64 in either tile.
static int split_for_mid_grid(const Problem &p, size_t workspace_bytes)
{
    if (!bf16_pingpong_eligible(p))
        return 0;
    const double kblocks = (double)p.batch * (double)(p.K / 64);
    const double t_128 = 3.0 + kblocks * 1.0;
    double best_t = t_128 * 0.92;                   // switch only for a clear gain
    if (wide_tile_wins(p) && !p.c_f32) {
        const double tiles = (double)(((p.M + 127) / 128) * ((p.N + 255) / 256));
        const double t_wide = 6.0 + kblocks * (0.62 + 0.21 * (tiles - 128.0) / 128.0);
        if (t_wide < best_t)
            best_t = t_wide;
    }
    return pingpong_split(p, workspace_bytes, kMaxSplit, best_t);
}

// At most 256 tiles of 128 x 128 on a B operand of 64 MB and more, other weights each time: a block of the 128-row kernel takes 0.575 us (0.4 from
// the caches; 57 B/ns of A and B together, however many blocks are requested ahead, and not for want of what memory gives all CUs), and 256 x 256 tiles pull half as much.  Other weights
// each time, 128 x 128 -> 256 x 256 with a split (us): 768 x 4096 x 11008 104 -> 77, 1024 x 4096 x 11008 107 -> 88, 1024 x 3072 x 12288 111 -> 81, 512 x
// 5120 x 7680 67 -> 55; of 45 sizes the slowest choice is 512 x 8192 x 8192, 73.8 -> 75.1.  Up to five slices: more take up to 1.3 times what the
// model says (512 x 4096 x 11008 with 8 74.6 us, with 6 60.4); and a row of tiles whose partial sums the allocation-free call can hold.  `split` is the 128-row kernel's.  Returns the other's, or 0.
static int split_for_streamed_b(const Problem &p, size_t workspace_bytes, int split)
{
    if (!in_16bit(p) || p.A_off || !bf16_pingpong_eligible(p) || (double)p.N * (double)p.K < 32.0e6)
        return 0;
    const int64_t tiles = ((p.M + 127) / 128) * ((p.N + 127) / 128), kblocks = p.batch * (p.K / 64);
    const int64_t most = BRGEMM_NOALLOC_SCRATCH_BYTES / ((int64_t)256 * p.N * (int64_t)sizeof(float));
    const double t = 5.5 + (double)((tiles * split + 255) / 256) * (double)((kblocks + split - 1) / split) * 0.575 +
                     (split > 1 ? 4.5 + (double)split * (double)p.M * (double)p.N * 4.0 / 4.0e6 : 0.0);
    return pingpong_split(p, workspace_bytes, most < 5 ? (int)most : 5, t * 0.92);
}

static int split_for_f32(const Problem &p, size_t workspace_bytes)
{
    const int64_t tiles = ((p.M + 127) / 128) * ((p.N + 127) / 128);
    const int64_t kblocks = p.K / 32;
    int best = 1;
    double best_t = 1e30;
    for (int s = 1; s <= kMaxSplit; ++s) {
        if (s > 1 && (kblocks / s < 1 || split_bytes(p, s) > workspace_bytes))
            continue;
        const double rounds = (double)((tiles * s + 255) / 256);
        const double per = (double)((kblocks + s - 1) / s);
        const double t_reduce = s > 1 ? 4.0 + (double)s * (double)p.M * (double)p.N * 8.0 / 3.0e6 : 0.0;
        const double t = 8.0 + rounds * per * 2.0 + t_reduce;
        if (t < best_t * 0.97) {
            best_t = t;
            best = s;
        }
    }
    return best;
}

// Time model of the general kernel, in microseconds beyond a launch, fitted to sweeps of all
// its tiles and splits 1-16 (51 x 7040 x 635 ... 3000^3, four layouts, odd and aligned rows).
// A step is 128 bytes of k for every group of the workgroup.  It costs `lone` with the chip
// nearly empty, `one` with a workgroup on every CU and `full` with two (16-bit and one-byte
// operands: L1 and LDS bytes; fp32, bound by the matrix pipe, gains nothing from a second),
// `mn` more for every m/n-contiguous operand (32 columns are half a cache line of a k-row),
// `edge` more where chunks straddle the end of such an operand and are shifted (the slowest
// workgroup counts), 0.15 over scattered tiles, a further round of workgroups `round` (first
// loads, epilogue), e.g. NT bf16 1000 x 2003 x 1500 takes 26.8 / 18.3 / 18.9 / 45.5 us as 128 x 128,
// 128 x 64, 64 x 64 and 32 x 32 tiles, 200 x 5000 x 1001 19.3 / 13.8 / 15.9 / 25.9, NN fp32 1024^3 74 / 42 / 26 / 38.
// A split adds a second launch and its partial tiles.
// However few its steps, a round of workgroups takes its first loads, the requests the 128-row
// tiles make ahead (in pairs, surplus ones included) and the epilogue: `least`, again with the chip
// nearly empty, a workgroup on every CU and two; `odd` times that where rows of C do not start on
// 16 bytes.  Fitted to 1,500 problems with K = 17 to 1500: the tile chosen takes 0.7 % more than the
// best one on average, 2.9 % without it.  33 x 65 x 40 (NT, bf16) took 5.5 us in a 128 x 64 tile and
// takes 4.4 in 64 x 64; 1001 x 1003 x 33 (NN, bf16) 9.0 and 6.5.  A step of fp32 takes longer than all that.
struct GenCost {
    int tile_m, tile_n, groups, per_cu;
    double round, lone, one, full, mn, edge, least[3], odd;
    double start, second, partial;      // beyond a launch; a split's second launch; TB/s of its partial tiles
};
static const GenCost gen_cost16[GEN_TILES] = {{128, 128, 1, 2, 0.3, 0.75, 1.05, 1.45, 0.05, 0.35, {3.3, 6.0, 9.9}, 1.35, 0.0, 5.0, 4.0},
                                              {128, 64, 1, 2, 0.3, 0.48, 0.56, 1.17, 0.05, 0.35, {1.5, 5.4, 6.3}, 1.16, 0.0, 5.0, 4.0},
                                              {64, 64, 2, 2, 0.3, 0.50, 0.72, 1.20, 0.05, 0.20, {0.5, 1.5, 3.7}, 1.15, 0.0, 5.0, 4.0},
                                              {32, 32, 8, 1, 1.8, 0.60, 0.75, 0.75, 0.15, 0.45, {}, 1.0, 0.0, 5.0, 4.0}};
static const GenCost gen_cost32[GEN_TILES] = {{128, 128, 1, 1, 0.3, 2.2, 2.3, 2.3, 0.1, 0.3, {}, 1.0, 0.0, 5.0, 4.0},
                                              {128, 64, 1, 1, 0.3, 1.2, 1.35, 1.35, 0.1, 0.25, {}, 1.0, 0.0, 5.0, 4.0},
                                              {64, 64, 2, 1, 0.3, 1.0, 1.40, 1.40, 0.05, 0.25, {}, 1.0, 0.0, 5.0, 4.0},
                                              {32, 32, 8, 1, 2.0, 1.3, 1.45, 1.45, 0.1, 0.4, {}, 1.0, 0.0, 5.0, 4.0}};
// The same where the wide tiles run as loading and multiplying waves (general_duty.hpp), fitted to
// 13,000 16-bit and 6,000 fp32 problems (16 x 64 x 130 ... 4200 x 6000 x 6000, four layouts, splits 1 to 6):
// the tile and split chosen take 1.1 % (fp32 0.3 %) more than the best measured on average, 4.2 % (1.2 %)
// with the constants above.  (`second` is 1 us above the fit, whose operands were in the caches: with
// weights from memory 5 x 1920 x 3006 takes 8.9 us in 32 x 32 tiles and 9.6 with the split it preferred.)
static const GenCost duty_cost16[GEN_TILES] = {{128, 128, 1, 2, 6.0, 0.40, 0.65, 1.31, 0.04, 0.02, {}, 1.0, 3.0, 2.0, 2.4},
                                               {128, 64, 1, 2, 3.7, 0.29, 0.40, 0.77, 0.03, 0.01, {}, 1.0, 1.8, 2.6, 2.3},
                                               {64, 64, 1, 2, 2.3, 0.17, 0.22, 0.49, 0.05, 0.01, {}, 1.0, 0.7, 3.5, 3.2},
                                               {32, 32, 8, 1, 2.5, 0.66, 0.96, 0.96, 0.16, 0.07, {}, 1.0, 0.4, 4.0, 4.0}};
static const GenCost duty_cost32[GEN_TILES] = {{128, 128, 1, 1, 0.8, 1.77, 1.98, 1.98, 0.08, 0.08, {}, 1.0, 3.2, 2.0, 2.3},
                                               {128, 64, 1, 2, 2.8, 0.90, 1.03, 1.93, 0.09, 0.07, {}, 1.0, 0.8, 2.6, 2.0},
                                               {64, 64, 1, 2, 2.4, 0.48, 0.52, 1.01, 0.06, 0.05, {}, 1.0, 0.0, 3.0, 1.9},
                                               {32, 32, 8, 1, 2.7, 1.26, 1.39, 1.39, 0.12, 0.17, {}, 1.0, 0.2, 4.0, 4.0}};
// The one-byte types, whose wide tiles are divided less often (duty_runs) and convert in the loading waves: fitted to 760 problems
// (4 to 60 sub-blocks, 0.3 to 1500 tiles of 128 x 128, four layouts).  The tile chosen takes 0.5 % (int8 0.2 %) more than the best; with the
// 16-bit constants it was 1.7 % and 1.3 %, and up to 1.5 times (FP8 TN 1922 x 1712 x 383: 12.2 us in 128 x 128, 15.9 in the 128 x 64 they prefer).
static const GenCost duty_cost_f8[GEN_TILES] = {{128, 128, 1, 2, 4.12, 0.49, 0.54, 1.61, 0.0, 0.15, {}, 1.0, 3.93, 2.0, 2.4},
                                                {128, 64, 1, 2, 2.82, 0.29, 0.26, 0.85, 0.03, 0.15, {}, 1.0, 2.03, 2.6, 2.3},
                                                {64, 64, 1, 2, 2.42, 0.16, 0.28, 0.48, 0.02, 0.02, {}, 1.0, 0.38, 3.5, 3.2},
                                                {32, 32, 8, 1, 2.93, 0.80, 0.80, 0.80, 0.09, 0.15, {}, 1.0, 0.0, 4.0, 4.0}};
static const GenCost duty_cost_s8[GEN_TILES] = {{128, 128, 1, 2, 5.89, 0.58, 0.71, 1.70, 0.0, 0.14, {}, 1.0, 3.11, 2.0, 2.4},
                                                {128, 64, 1, 2, 3.70, 0.42, 0.52, 1.17, 0.0, 0.09, {}, 1.0, 1.32, 2.6, 2.3},
                                                {64, 64, 1, 2, 1.98, 0.24, 0.32, 0.72, 0.04, 0.05, {}, 1.0, 0.0, 3.5, 3.2},
                                                {32, 32, 8, 1, 2.46, 0.92, 1.30, 1.30, 0.41, 0.23, {}, 1.0, 0.0, 4.0, 4.0}};

static const GenCost &general_cost(const Problem &p, int form, bool divided)
{
    if (divided)
        return p.in_s8 ? duty_cost_s8[form] : in_8bit(p) ? duty_cost_f8[form] : in_16bit(p) ? duty_cost16[form] : duty_cost32[form];
    return (in_16bit(p) || in_8bit(p)) ? gen_cost16[form] : gen_cost32[form];
}

// What does not change from split to split, for the plan's loop over them.
struct GenModel {
    const GenCost *c;
    int64_t tiles, steps;       // steps: sub-blocks of a tile, batch included
    double full, lone, one, partial_us, odd;
    int slot_shift;             // 256 or 512 workgroups at once

    GenModel(const Problem &p, int form, bool divided) : GenModel(p, general_cost(p, form, divided)) {}
    GenModel(const Problem &p, const GenCost &cost) : c(&cost)
    {
        tiles = ((p.M + c->tile_m - 1) / c->tile_m) * ((p.N + c->tile_n - 1) / c->tile_n) * p.nmat;
        const int sub = p.in_s8 ? 128 : (in_16bit(p) || in_8bit(p)) ? 64 : 32;
        steps = p.batch * ((p.K + sub - 1) / sub);
        const int chunk = in_16bit(p) ? 8 : p.in_s8 ? 16 : p.in_f8 ? 8 : 4;
        const bool a_mn = p.transA == 1, b_mn = p.transB == 0 && !p.b_packed;
        const double extra = (a_mn + b_mn) * c->mn + ((a_mn && p.M % chunk) || (b_mn && p.N % chunk) ? c->edge : 0.0) +
                             (p.A_off ? 0.15 : 0.0);
        full = c->full + extra;
        lone = c->lone + extra;
        one = c->one + extra;
        partial_us = (double)p.M * (double)p.N * 4.0 / (c->partial * 1.0e6);
        slot_shift = c->per_cu == 2 ? 9 : 8;
        odd = (p.ldc & 3) || ((uintptr_t)p.C & 15) ? c->odd : 1.0;
    }
    // Beyond the time of its kernel a split costs a second launch and its partial tiles.
    double split_us(int split) const { return split > 1 ? c->second + (double)split * partial_us : 0.0; }

    // floors: with the least time of a round (fitted to unsplit problems; the constants that small
    // grids are compared with were fitted without it)
    double us(int split, bool floors) const
    {
        const double per = (double)(((steps + split - 1) / split + c->groups - 1) / c->groups);
        const int64_t wgs = tiles * split, rounds = wgs >> slot_shift, rest = wgs - (rounds << slot_shift);
        const double part = (double)rest / 256.0;
        auto at_least = [&](double t, double least) { return floors && split == 1 && t < least * odd ? least * odd : t; };
        double t = (double)rounds * at_least(c->round + per * (c->per_cu == 2 ? full : one), c->least[2]);
        if (rest > 256)
            t += at_least(c->round + per * full, c->least[1] + (c->least[2] - c->least[1]) * (part - 1.0));
        else if (rest > 0)
            t += at_least(c->round + per * (lone + (one - lone) * part), c->least[0] + (c->least[1] - c->least[0]) * part);
        return t - c->round + c->start + split_us(split);   // the first round's is part of the launch
    }
};

// A 16-bit problem whose rows the tuned kernels can read but whose K ends inside a block of 64.  Shorter reductions stay
// with the general kernel: the incomplete block is not overlapped with anything (the line itself is not measured).
static bool ends_in_a_block(const Problem &p)
{
    return p.K % 64 != 0 && p.K >= 512 && p.batch == 1 && !p.A_off && bf16_rows_eligible(p);
}

// Beyond a launch, in microseconds: the 256 x 256 kernel (one workgroup on a CU; a last round of few tiles runs at a higher clock) and
// the general kernel's undivided 128 x 128 tile on rows that the tuned kernels can read (two).  Fitted to 235 problems of more
// than 512 tiles of 128 x 128, K = 513 to 5000: the faster one by these takes 0.7 % more than the faster one measured.  Always the first
// took 4.3 % more: it has a quarter of the tiles, and of a last round of few tiles as much is paid as of a whole one
// (TT 2384 x 6728 x 835, 270 tiles: 67.5 us, in general tiles 47.7; 4096 x 4096 x 4000, 256: 98.5, 153).  Rows of C off 16 bytes cost
// it 9 (fp32) or 14 us more a round (NT 1498 x 13315 x 656 92.0, 50.7).
static double pingpong_us(const Problem &p)
{
    const int64_t tiles = ((p.M + 255) / 256) * ((p.N + 255) / 256) * p.nmat;
    const double per = (double)((p.K + 63) / 64), rounds = (double)(tiles / 256), part = (double)(tiles % 256) / 256.0;
    const double odd = !((p.ldc & 3) || ((uintptr_t)p.C & 15)) ? 0.0 : p.c_f32 ? 9.0 : 14.0;      // C stored an element at a time
    return 0.3 + rounds * (18.7 + odd + per * 1.313) + (part > 0.0 ? 8.2 + odd + 10.5 * part + per * (1.114 + 0.193 * part) : 0.0);
}
static double readable_rows_us(const Problem &p)
{
    const int64_t tiles = ((p.M + 127) / 128) * ((p.N + 127) / 128) * p.nmat, rest = tiles % 512;
    const double per = (double)((p.K + 63) / 64), part = (double)rest / 256.0;
    return 0.1 + (double)(tiles / 512) * (4.7 + per * 1.115) +
           (rest == 0 ? 0.0 : 4.7 + per * (rest > 256 ? 1.115 : 0.433 + 0.130 * part));
}

// Which tuned kernel takes such a problem: by grid as the table above does it, the 48-column weight stream
// included.  In the general kernel's own tiles -> now (us): 4096 x
// 4096 x 4000 NT 153 -> 98.5 (K = 4096: 95), NN 157 -> 99, 2048 x 4096 x 4000 NT 80 -> 63, 2048 x 2048 x 2000 NN 27.8 ->
// 23.3, 128 x 11008 x 4000 NT 28.1 -> 27.0.
TailKernel tail_kernel(const Problem &p, int split)
{
    if (!ends_in_a_block(p))
        return TAIL_NONE;
    const int64_t tm = (p.M + 127) / 128, tn = (p.N + 127) / 128, tiles = tm * tn * p.nmat, narrow = (p.N + 47) / 48;
    if (split == 1 && p.transA == 0 && p.transB == 1 && !p.b_packed && p.M > 80 && p.M <= 128 && p.nmat == 1 && narrow >= 192 && narrow <= 256)
        return TAIL_NARROW;
    if (tiles * split <= 256)
        return TAIL_128;
    if (split > 1)
        return TAIL_NONE;
    if (tm * ((p.N + 255) / 256) * p.nmat <= 256)
        return TAIL_WIDE;
    return tiles > 512 && pingpong_us(p) < readable_rows_us(p) ? TAIL_PINGPONG : TAIL_NONE;
}

// Time of that kernel beyond a launch, in microseconds.
static double tail_us(const Problem &p, TailKernel k, int split)
{
    const int64_t tm = (p.M + 127) / 128, tn = (p.N + 127) / 128;
    const double per = (double)(((p.K + 63) / 64 + split - 1) / split);
    const double k_rows = (p.transA == 0) + (p.transB == 1 && !p.b_packed);
    const double extra = split > 1 ? 3.0 + (double)split * (double)p.M * (double)p.N * 4.0 / 2.4e6 : 0.0;
    switch (k) {
    case TAIL_NARROW: return 2.0 + per * 0.31;
    case TAIL_128:          // (a row along k whose 128 bytes straddle two cache lines: 2048 x 2048 x 2000 NT 26.6, NN 23.3)
        return 2.8 + per * (0.36 + 0.04 * k_rows + 0.14 * (double)(tm * tn * p.nmat * split) / 256.0) + extra;
    case TAIL_WIDE: return 5.0 + per * (0.64 + 0.21 * ((double)(tm * ((p.N + 255) / 256) * p.nmat) - 128.0) / 128.0);
    default: return pingpong_us(p);
    }
}

hipError_t launch_tail(const Problem &p)
{
    const TailKernel k = tail_kernel(p, p.split);
    return k == TAIL_PINGPONG ? launch_pingpong_tail(p) : launch_stream_tail(p, k);
}

// Copying `bytes` of operands and multiplying the copies in 256 x 256 tiles, against the general kernel's 128 x 128 tiles
// (whose rows off 16 bytes take 1.136 of the model above, fitted to all alignments).  Fitted to 134 problems of 513 to 1,800 tiles of
// 128 x 128, K = 513 to 6500: the faster one by these takes 0.5 % more than the faster one measured; 5 of the copied are 3 to 19 %
// slower copied.  The rounds decide: NN 1503 x 9730 x 625, 234 tiles of 256 x 256, 43.7 us in general tiles and 60.3 copied; NT 4095^3,
// 256, 201 and 151.  Asked where the plan, which does not count the copies, picked 128 x 128.
bool realign_pays(const Problem &p, size_t bytes)
{
    return 2.0 * (double)bytes / 4.0e6 + 6.2 + pingpong_us(p) < 1.136 * GenModel(p, GEN_128, duty_eligible(p)).us(1, true);
}

// Tile and reduction split of the general kernel.  A split whose partial sums exceed what
// the allocation-free entry point can hold is not taken, so that call accepts every problem
// it would run unsplit.  The loop over splits ends where one cannot win by its second launch and
// its partial tiles alone, which for most problems is before the first (a call of a few
// elements is bound by its host side: trying all 16 splits of four tiles took 1.0 to 1.3 us of it,
// this takes 0.1).
static void plan_general(const Problem &p, size_t workspace_bytes, bool may_split, int fixed_split, int fixed_form, Plan *out)
{
    const size_t room = workspace_bytes < BRGEMM_NOALLOC_SCRATCH_BYTES ? workspace_bytes : BRGEMM_NOALLOC_SCRATCH_BYTES;
    const int first = fixed_split > 0 ? fixed_split : 1, last = fixed_split > 0 ? fixed_split : may_split ? kMaxSplit : 1;
    double best_t = 1e30;
    const bool divided = duty_eligible(p);
    for (int f = 0; f < GEN_TILES; ++f) {
        if (fixed_form >= 0 && f != fixed_form)
            continue;
        const GenModel model(p, f, divided);
        const bool readable = f == GEN_128 && model.tiles > 512 && ends_in_a_block(p);
        const int least_steps = divided && f != GEN_32 ? 4 : model.c->groups;      // of a slice
        for (int s = first; s <= last; ++s) {
            if (fixed_split <= 0 && s > 1 &&
                (model.split_us(s) >= best_t * 0.97 || (model.steps + s - 1) / s < least_steps || split_bytes(p, s) > room))
                break;
            const TailKernel k = f == GEN_128 ? tail_kernel(p, s) : TAIL_NONE;
            const double t = k != TAIL_NONE ? tail_us(p, k, s) : readable && s == 1 ? readable_rows_us(p) : model.us(s, true);
            if (t < best_t * 0.97) {
                best_t = t;
                out->form = f;
                out->split = s;
            }
        }
    }
    if (general_short_runs(p))
        out->form = GEN_64;                         // the one tile that gathers its chunks
}

// Where the short kernel beats every tile of the general one: up to K = 16 at every size measured
// (1 x 10001 to 4001 x 4003, six operand types, four layouts: 0.4 to 0.95 of the best tile's time); with
// K = 17 to 32 always in fp32 (4001 x 4003: 0.66 to 0.84), and in the narrower types, whose own
// instruction needs one step for all of it, up to so many 64 x 64 tiles (16-bit and FP8, K up to 24,
// 1,500 to 2,500 tiles: 0.69 to 0.92 of the best, K = 25 to 32, 625: 0.67 to 0.87, 814: 0.88 to 1.07; int8
// at 650 0.76 to 0.98, at 1,500 and more 0.73 to 1.22).  A batch-reduce of one tile is such a product at
// an offset: 5 x 7 to 4001 x 4003 of bf16 and fp32, NN, NT and TT, 0.53 to 0.91 of the tiles' time (bf16
// 64 x 64, K below 16, 5.2 -> 4.1 us; fp32 2001 x 2003, K = 16 to 32, 14.5 -> 9.0).
static bool short_wins(const Problem &p)
{
    if (p.batch != 1 || p.K > kMaxShort)
        return false;
    if (p.K <= 16 || !(in_16bit(p) || in_8bit(p)))
        return true;
    return ((p.M + 63) / 64) * ((p.N + 63) / 64) * p.nmat <= (p.in_s8 || p.K > 24 ? 700 : 2560);
}

int choose_plan(const Problem &p, size_t workspace_bytes, int forced_variant, int forced_split, int forced_form, Plan *out)
{
    Plan plan{V_GENERIC, 1, -1};
    // A batched call (nmat matrices) multiplies the tile count and never splits.
    const bool single = p.nmat == 1 && !p.in_s8;     // int8 sums are not split (the reduction adds floats)
    const int skinny_bm = p.M <= 32 ? 32 : p.M <= 64 ? 64 : 128;
    if (p.M <= 128 && bf16_stream_eligible(p, skinny_bm)) {
        // Few rows of A: the time goes into streaming B once.
        plan.variant = skinny_bm == 32 ? V_BF16_STREAM32 : skinny_bm == 64 ? V_BF16_STREAM64 : V_BF16_STREAM128;
        plan.split = single ? split_for_stream(p, skinny_bm, workspace_bytes) : 1;
    } else if (bf16_mfma_eligible(p)) {
        // 128x128 tiles while all of them are resident at once (two workgroups per CU:
        // 512), 256x256 tiles beyond that (measured crossover on squares: 2816 -> 3072).
        const int64_t t128 = ((p.M + 127) / 128) * ((p.N + 127) / 128) * p.nmat;
        if (t128 > 512) {
            plan.variant = V_BF16_PP256;
        } else {
            // Up to 256 tiles leave at most one workgroup per CU: a streaming kernel, its
            // tile height by how many workgroups that puts on the chip; between 257 and 512
            // one round of 128 x 256 tiles where that fits (wide_tile_wins), else the two-stage kernel,
            // two of whose workgroups share a CU, or 256 x 256 tiles with a split.
            if (t128 <= 256 && bf16_stream_eligible(p, 128)) {
                int bm = 128, split = 1;
                plan_small_grid(p, workspace_bytes, single, &bm, &split);
                plan.variant = bm == 32 ? V_BF16_STREAM32 : bm == 64 ? V_BF16_STREAM64 : V_BF16_STREAM128;
                plan.split = split;
                const int pp_split = single && bm == 128 ? split_for_streamed_b(p, workspace_bytes, split) : 0;
                if (pp_split > 0) {
                    plan.variant = V_BF16_PP256;
                    plan.split = pp_split;
                    plan.displaced = split;
                }
            } else {
                const int pp_split = (single && !p.in_f8) ? split_for_mid_grid(p, workspace_bytes) : 0;
                if (pp_split > 0) {
                    plan.variant = V_BF16_PP256;
                    plan.split = pp_split;
                } else {
                    plan.variant = (p.in_f8 && bf16_stream_eligible(p, 128)) ? V_BF16_STREAM128 : V_BF16_128x128;
                    plan.split = single && !wide_tile_wins(p) ? split_for_small_grid(p, workspace_bytes) : 1;
                }
            }
        }
    }
    if (f32_mfma_eligible(p)) {
        plan.variant = V_F32_128x128;
        plan.split = single ? split_for_f32(p, workspace_bytes) : 1;
    }
    if (forced_variant >= 0) {
        if (forced_variant >= V_COUNT || !variant_eligible(forced_variant, p))
            return BRGEMM_INVALID_ARG;
        if (plan.displaced > 0 && forced_variant != V_BF16_PP256) {
            plan.split = plan.displaced;            // not a split of other tiles
            plan.displaced = 0;
        }
        plan.variant = forced_variant;
    }
    if (forced_split > 1 && !single)
        return BRGEMM_INVALID_ARG;
    if (plan.variant == V_GENERIC && forced_form < 0 && forced_split <= 1 && short_wins(p))
        forced_form = FORM_SHORT;
    if (forced_form >= 0) {
        const bool unsplit = plan.variant != V_GENERIC || forced_form == FORM_SHORT;
        if (!form_eligible(forced_form, plan.variant, p) || (unsplit && forced_split > 1))
            return BRGEMM_INVALID_ARG;
        plan.split = 1;
        plan.form = forced_form;
    }
    if (plan.variant == V_GENERIC && forced_form != FORM_SHORT)
        plan_general(p, workspace_bytes, single, forced_split, forced_form, &plan);
    if (forced_split > 0) {
        plan.split = forced_split;
        plan.displaced = 0;                         // (its own split was bounded by the library's buffer)
        if (split_bytes(p, plan.split) > workspace_bytes)
            return BRGEMM_WORKSPACE_TOO_SMALL;
    }
    *out = plan;
    return BRGEMM_OK;
}

// Small grids: the tuned kernels' 128-column tiles leave most of the chip without work, and a
// split over workgroups costs partial tiles and a second launch.  The general kernel's 64-
// and 32-wide tiles put more workgroups on the chip and divide the work of ONE workgroup between its waves (the
// 32-wide ones its reduction).  This compares the two by time models (microseconds beyond a
// launch; constants of the tuned kernels from the same sweeps: a k-block costs a workgroup
// 0.30 / 0.35 / 0.42 us at 32 / 64 / 128 rows plus 1.2 us of deeper prologue at 128, up to
// twice that where every block is a scattered tile; fp32 2.0 us).  Measured, tuned -> this: bf16
// 512 x 512 x 2048 14.4 -> 7.6 us, 128 x 2048 x 1024 10.8 -> 6.1, 512 x 512 x 4096 12.8 -> 10.6;
// fp32 256^3 10.7 -> 6.1, 512^3 15.5 -> 7.7, 1024 x 1024 x 256 20.9 -> 10.4.  The models are those of the undivided tiles: where the
// 64 x 64 tile runs divided (duty_runs) it is faster than this says.  fp32 1024^3: 30.0 us with split 4, 24.5 in 64 x 64 tiles, whose sums are
// two chains where the split has four: 4.1e-7 from 64 bits against 2.9e-7.  Plain 16-bit products go on to prefer_stream_forms.  `plan` is the table's.
static void prefer_stream_forms(const Problem &p, size_t workspace_bytes, Plan *io);

static void prefer_other_forms(const Problem &p, size_t workspace_bytes, Plan *io)
{
    const Plan plan = *io;
    // The 48-column form of the 128-row streaming kernel: 192 to 256 of its tiles put a whole
    // weight stream on the chip in one round, without a split.  81 to 128 rows, split plan ->
    // this, weights from memory: 128 x 11008 x 4096 31.4 -> 28.3 us (from the last-level cache 23.6 -> 23.5),
    // 128 x 9216 x 2048 16.3 -> 13.8, 96 x 12288 x 4096 31.1 -> 29.0; with 125 tiles (N = 6000) 18.1 -> 21.9, and
    // at 64 rows level.  Only a split plan is replaced, so a call without a workspace keeps 128 columns.
    const int64_t narrow = (p.N + 47) / 48;
    if (plan.split > 1 && form_eligible(FORM_NARROW, plan.variant, p) && p.M > 80 && p.M <= 128 && p.nmat == 1 &&
        narrow >= 192 && narrow <= 256) {
        *io = Plan{plan.variant, 1, FORM_NARROW};
        return;
    }
    if (plan.variant == V_GENERIC || !form_eligible(GEN_32, plan.variant, p))
        return;
    // (Few rows of A on a large weight matrix: its stream bounds every plan, and the table's splits and this choice are fitted to that.  16 x
    // 11008 x 4096: 21.8 us with split 5, 22.4 as 172 tiles of 64 x 64; 192 x 4096 x 4096 17.3 with split 4, 18.5; 52 x 4096 x 4096 10.6 in
    // 32 x 32 tiles, 12.0 with split 6.  Packed B the other way, the split against 32 x 32 tiles: 11.5 and 13.2, 16 x 4096 x 4096 8.4 and 12.4, eight wider or
    // longer ones choose the split anyway.  So with 16-bit C the table's plan stays; an fp32 C keeps the 32 x 32 tiles' eight chains,
    // whose sums are the closer ones: 52 rows 1.37e-7 from 64 bits against 1.55e-7, 16 rows both 1.38e-7.)
    const bool weights = p.M <= 256 && 2.0 * (double)p.N * (double)p.K > 32.0e6;
    const bool streams = in_16bit(p) && p.batch == 1 && !p.A_off && !weights;
    if (weights && p.b_packed && !p.c_f32)
        return;
    if (streams && !p.c_f32) {
        prefer_stream_forms(p, workspace_bytes, io);
        return;
    }
    const double split_us = plan.split > 1 ? (p.A_off ? 3.2 : 4.2) + (double)plan.split * (double)p.M * (double)p.N * 4.0 / 4.2e6 : 0.0;
    double t;
    if (plan.variant == V_F32_128x128) {
        const int64_t wgs = ((p.M + 127) / 128) * ((p.N + 127) / 128) * p.nmat * plan.split;
        t = (double)((wgs + 255) / 256) * (double)((p.K / 32 + plan.split - 1) / plan.split) * 2.0;
    } else {
        const int bm = plan.variant == V_BF16_STREAM32 ? 32 : plan.variant == V_BF16_STREAM64 ? 64 : 128;
        const int64_t kblocks = p.batch * (p.K / (p.in_s8 ? 128 : 64));
        const int64_t wgs = ((p.M + bm - 1) / bm) * ((p.N + 127) / 128) * p.nmat * plan.split;
        const int64_t at_once = bm == 128 ? 256 : 512;
        const double block = (bm == 32 ? 0.30 : bm == 64 ? 0.35 : 0.42) * (p.A_off && p.K < 192 ? 1.0 + (192.0 - (double)p.K) / 128.0 : 1.0);
        t = (double)((wgs + at_once - 1) / at_once) * (double)((kblocks + plan.split - 1) / plan.split) * block +
            (bm == 128 ? 1.2 : 0.0);
    }
    t += split_us;
    int best = -1;
    double best_t = (4.5 + t) * 0.93 - 4.8;                     // a clear gain of the whole call
    for (int f = GEN_64; f <= GEN_32; ++f) {
        const double g = GenModel(p, f, false).us(1, false);
        if (g < best_t) {
            best_t = g;
            best = f;
        }
    }
    if (best >= 0)
        *io = Plan{p.nmat > 1 ? V_GENERIC : plan.variant, 1, best};  // the variant's reduced-tile form
    if (streams && io->form != GEN_64)
        prefer_stream_forms(p, workspace_bytes, io);
}

// (Sums that stay in fp32 start from the choice above and leave it only for tiles whose sums are closer to the exact one: the
// 32 x 32 tile's eight chains stay where the 32 x 128 kernel's one would be faster.)
// The plan of a plain 16-bit product that the table gives to a streaming kernel: its kernel and split, or the general path's
// 32 x 32, 64 x 64 (split or not) or 128 x 64 tiles, by one time model.  Constants fitted to 1,500 problems (1 x 64 x 64 ... 3000 x 6000 x 6000, four
// layouts, operands from the last-level cache) with all splits measured, 23,000 times in all; a kernel's mean error is 4 to 5 %.
// The plan chosen took 1.7 % more than the best one measured, the table's with the undivided tiles' constants 4.1 % (14 % where it was
// 128 x 128): NT 232 x 3064 x 1984 16.0 us in 128 x 128 tiles with split 4, 11.0 in 64 x 64; TN 128 x 320 x 5248 16.4 in 32 x 32, 8.9 in 64 x 64 with split 8.
static const GenCost stream_cost[] = {{32, 32, 8, 1, 1.77, 0.63, 1.01, 1.01, 0.08, 0.0, {}, 1.0, -0.99, 4.0, 4.0},
                                      {64, 64, 1, 2, 1.64, 0.19, 0.23, 0.40, 0.01, 0.0, {}, 1.0, -0.04, 2.1, 3.5},
                                      {128, 64, 1, 2, 0.03, 0.30, 0.37, 0.62, 0.0, 0.0, {}, 1.0, 0.56, 2.0, 2.4},
                                      {32, 128, 1, 2, 1.95, 0.28, 0.32, 0.46, 0.0, 0.0, {}, 1.0, -0.55, 2.1, 5.6},
                                      {64, 128, 1, 2, 0.0, 0.36, 0.44, 0.65, 0.01, 0.0, {}, 1.0, -0.61, 1.9, 2.8},
                                      {128, 128, 1, 1, 0.57, 0.35, 0.45, 0.45, 0.01, 0.0, {}, 1.0, 1.47, 1.4, 2.3}};
enum { SC_32, SC_64, SC_MID, SC_S32, SC_S64, SC_S128 };

// Instead of the full tiles of a plan, those that stream_tile_instead names, or -1.
static int instead_of_full_tiles(const Problem &p, const Plan &plan)
{
    if (plan.form >= 0 || (plan.variant != V_BF16_STREAM32 && plan.variant != V_BF16_STREAM64))
        return -1;
    return stream_tile_instead(p, plan.variant == V_BF16_STREAM32 ? 32 : 64, plan.split);
}

void prefer_small_tiles(const Problem &p, size_t workspace_bytes, Plan *io)
{
    prefer_other_forms(p, workspace_bytes, io);
    const int tile = instead_of_full_tiles(p, *io);
    if (tile >= 0)
        *io = Plan{p.nmat > 1 ? (int)V_GENERIC : io->variant, 1, tile};
}

static void prefer_stream_forms(const Problem &p, size_t workspace_bytes, Plan *io)
{
    const int own = instead_of_full_tiles(p, *io);
    const int table = io->form == GEN_32 ? SC_32 : own == GEN_64 ? SC_64 : own == GEN_MID ? SC_MID
                      : io->variant == V_BF16_STREAM32 ? SC_S32 : io->variant == V_BF16_STREAM64 ? SC_S64 : SC_S128;
    // (a launch; no kernel streams its operands faster than memory does)
    const double floor_us = 4.9, launch_us = 4.3;
    const double stream_us = 2.0 * ((double)p.M + (double)p.N) * (double)p.K * (double)p.nmat / 5.5e6;
    auto call_us = [&](const GenModel &m, int split) {
        const double t = m.us(split, false), kernel = t - m.split_us(split);
        const double all = launch_us + t + (kernel < stream_us ? stream_us - kernel : 0.0);
        return all < floor_us ? floor_us : all;
    };
    const size_t room = workspace_bytes < BRGEMM_NOALLOC_SCRATCH_BYTES ? workspace_bytes : BRGEMM_NOALLOC_SCRATCH_BYTES;
    double best_t = call_us(GenModel(p, stream_cost[table]), io->split) * 0.93;     // a clear gain
    Plan best = *io;
    static const int forms[] = {GEN_32, GEN_64, GEN_MID};
    for (int f = p.c_f32 ? SC_64 : SC_32; f <= SC_MID; ++f) {
        const GenModel model(p, stream_cost[f]);
        const int last = f == SC_32 || p.nmat > 1 ? 1 : kMaxSplit;
        for (int s = 1; s <= last; ++s) {
            if (s > 1 && ((model.steps + s - 1) / s < 4 || split_bytes(p, s) > room || launch_us + model.split_us(s) >= best_t))
                break;
            if (f == SC_MID && (p.c_f32 || s > 1) && model.tiles * s > 256)
                break;                              // (registers for one workgroup on a CU)
            const double t = call_us(model, s);
            if (t < best_t * (s > 1 ? 0.98 : 1.0)) {
                best_t = t;
                best = Plan{s > 1 || f == SC_MID || p.nmat > 1 ? (int)V_GENERIC : io->variant, s, forms[f]};
            }
        }
    }
    *io = best;
}

hipError_t launch_variant(int v, const Problem &p)
{
    if (p.form == FORM_NARROW)
        return launch_bf16_stream_narrow(p);
    if (p.form == FORM_SHORT)
        return general_launch_short(p);
    if (p.form >= 0)
        v = V_GENERIC;                              // a tuned variant's reduced-tile form
    switch (v) {
    case V_GENERIC:
        if (!general_short_runs(p) && !general_offsets_fit(p, p.form))
            return general_launch_far(p, p.form);
        return p.A_off ? general_launch_offsets(p, p.form)
               : in_16bit(p) ? general_launch_half(p, p.form)
               : in_8bit(p) ? general_launch_bytes(p, p.form) : general_launch_f32(p, p.form);
    case V_BF16_128x128: return launch_bf16_128x128(p);
    case V_BF16_PP256: return launch_bf16_pingpong(p);
    case V_F32_128x128: return launch_f32_128x128(p);
    case V_BF16_STREAM32: return launch_bf16_stream(p, 32);
    case V_BF16_STREAM64: return launch_bf16_stream(p, 64);
    case V_BF16_STREAM128: return launch_bf16_stream(p, 128);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace brg
