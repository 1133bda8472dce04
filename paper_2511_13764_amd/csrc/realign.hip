// Large 16-bit products whose rows start off 16 bytes: the operands are copied into the caller's
// workspace with rows on whole cache lines, and the 256 x 256 kernel takes the copies.
//
// What it is for: the general kernel pulls such rows through registers at 53-80 B/ns per CU and
// multiplies at about 0.7 PFLOP/s; the 256 x 256 kernel reaches 1.4, and the copy moves each operand
// twice.  The copy is bound by memory and the caches (16 bytes per lane, one launch for both operands).
// Measured, in the general kernel's tiles -> this (us): NT 4095^3 201 -> 151, 4000 x
// 4000 x 2500 (ld 2501) 134 -> 89, 4096 x 11008 x 1001 159 -> 107; NN 4095^3 209 -> 154, 3500 x 3500 x 2000 93 -> 73; TN 4095^3 241 -> 160.
#include "bf16_tiles.hpp"

namespace brg {

namespace {

struct RealignArgs {
    const uint16_t *src[2];
    uint16_t *dst[2];
    int64_t ld[2], dst_ld[2];
    uint32_t cols[2], chunks[2], total[2];      // chunks: of 8 values, in a row of the copy
};

// One 16-byte chunk of the copy per thread, zeros past the row's end (cols >= 512).
__global__ void __launch_bounds__(256)
realign_kernel(RealignArgs a)
{
    const int o = blockIdx.y;
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= a.total[o])
        return;
    const uint32_t row = i / a.chunks[o], c = i - row * a.chunks[o];
    const int over = (int)(c * 8 + 8) - (int)a.cols[o];
    const uint16_t *src = a.src[o] + (int64_t)row * a.ld[o] + c * 8 - (over > 0 ? over : 0);
    s16x8 v = *(const s16x8_any2 *)src;
    if (over > 0)
        v = drop16(v, over < 8 ? over : 8);
    *(s16x8 *)(a.dst[o] + (int64_t)row * a.dst_ld[o] + c * 8) = v;
}

struct Stored { int64_t rows, cols, ld; bool copy; };

// An operand as it is stored, and whether the 16-byte loads of the tuned kernels can read it.
Stored stored(const void *ptr, int64_t rows, int64_t cols, int64_t ld, bool mn)
{
    return Stored{rows, cols, ld, ((uintptr_t)ptr & 15) != 0 || (ld & 7) != 0 || (mn && (cols & 7) != 0)};
}
Stored stored_a(const Problem &p) { return p.transA ? stored(p.A, p.K, p.M, p.lda, true) : stored(p.A, p.M, p.K, p.lda, false); }
Stored stored_b(const Problem &p) { return p.transB ? stored(p.B, p.N, p.K, p.ldb, false) : stored(p.B, p.K, p.N, p.ldb, true); }

// Whole cache lines.
int64_t copy_ld(const Stored &s) { return (s.cols + 63) / 64 * 64; }
size_t copy_bytes(const Stored &s) { return s.copy ? ((size_t)s.rows * (size_t)copy_ld(s) * 2 + 255) / 256 * 256 : 0; }

}  // namespace

// More 128 x 128 tiles than the chip holds at once (the 256 x 256 kernel's grids), the copies fit the
// workspace, and by the time models the faster kernel saves more than the copies take.  Asked at the launch of the general
// path's 128 x 128 form: the plan does not count the copies, so a call that it gives other tiles is not copied.
bool realign_wins(const Problem &p)
{
    if (!in_16bit(p) || p.batch != 1 || p.A_off || p.b_packed || p.nmat != 1 || p.split != 1 || !p.scratch || p.K < 512)
        return false;
    if (((p.M + 127) / 128) * ((p.N + 127) / 128) <= 512 || p.M < 512 || p.N < 512 || p.M >= (1 << 22) || p.N >= (1 << 22) || p.K >= (1 << 22) ||
        p.lda >= (1 << 22) || p.ldb >= (1 << 22) || p.M * p.N >= ((int64_t)1 << 40))
        return false;
    const Stored a = stored_a(p), b = stored_b(p);
    const size_t bytes = copy_bytes(a) + copy_bytes(b);
    if (bytes == 0 || bytes > p.scratch_bytes || bytes > (size_t)kMaxSplit * (size_t)p.M * (size_t)p.N * sizeof(float) ||
        bytes >= ((size_t)1 << 34))
        return false;
    return realign_pays(p, bytes);
}

hipError_t launch_realigned(const Problem &p)
{
    const Stored s[2] = {stored_a(p), stored_b(p)};
    const void *ptr[2] = {p.A, p.B};
    char *room = (char *)p.scratch;
    Problem q = p;
    RealignArgs a{};
    unsigned n = 0;
    uint32_t blocks = 0;
    for (int o = 0; o < 2; ++o) {
        if (!s[o].copy)
            continue;
        a.src[n] = (const uint16_t *)ptr[o];
        a.dst[n] = (uint16_t *)room;
        a.ld[n] = s[o].ld;
        a.dst_ld[n] = copy_ld(s[o]);
        a.cols[n] = (uint32_t)s[o].cols;
        a.chunks[n] = (uint32_t)(copy_ld(s[o]) / 8);
        a.total[n] = (uint32_t)((uint64_t)s[o].rows * a.chunks[n]);
        blocks = blocks > (a.total[n] + 255) / 256 ? blocks : (a.total[n] + 255) / 256;
        (o ? q.B : q.A) = room;
        (o ? q.ldb : q.lda) = copy_ld(s[o]);
        room += copy_bytes(s[o]);
        ++n;
    }
    hipLaunchKernelGGL(realign_kernel, dim3(blocks, n), dim3(256), 0, p.stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return q.K % 64 ? launch_pingpong_tail(q) : launch_bf16_pingpong(q);
}

}  // namespace brg
