// Short reductions (K <= 32) of the general path: any size, alignment, layout and operand type.
// Operands are widened exactly to fp32 (int8 too: 32 products of 2^14 stay far below 2^24) and
// multiplied on the fp32 matrix instruction.
//
// What bounds it: nothing but a chain of latencies on a small C, the stores of C on a large
// one.  So there is one request of everything, one barrier, and no staging of C: with B as the
// first operand a lane holds four consecutive columns of a row and stores them as they are.
// The tiles of general.hpp, which widen nothing but make four barriers, requests ahead and 128
// bytes of k out of whatever there is, take (us, theirs -> this): bf16 NN 5 x 7 x 5 5.6 -> 3.8, 33 x 65 x 16
// 4.8 -> 3.9, 1000 x 1000 x 16 7.1 -> 4.3, 4001 x 4003 x 5 44.5 -> 17.2 (32 MB of C: 6.4 at the
// rate of a copy); fp32 4000 x 4000 x 16 28.5 -> 17.3; int8 NT 300 x 300 x 8 6.7 -> 4.1.
#include "general.hpp"

namespace brg {

namespace {

constexpr int ST = 64;                  // tile edge (M and N); four wavefronts of 32 x 32

struct ShortArgs {
    int64_t M, N, K, lda, ldb, ms_a, ms_b, ms_c;
    const char *A, *B;
    const int64_t *A_off, *B_off;       // a batch-reduce of one tile: where it starts, or nullptr
    int transA, transB, b_packed;
    Epilogue epi;
};

template <int KIND>
__device__ __forceinline__ float widen(const char *p, int64_t i)
{
    if constexpr (KIND == KIND_BF16)
        return bf16_to_f32(((const uint16_t *)p)[i]);
    else if constexpr (KIND == KIND_F16)
        return f16_to_f32(((const uint16_t *)p)[i]);
    else if constexpr (KIND == KIND_S8)
        return (float)((const int8_t *)p)[i];
    else if constexpr (KIND == KIND_F8)
        return __builtin_amdgcn_cvt_f32_fp8((int)((const uint8_t *)p)[i], 0);
    else if constexpr (KIND == KIND_BF8)
        return __builtin_amdgcn_cvt_f32_bf8((int)((const uint8_t *)p)[i], 0);
    else
        return ((const float *)p)[i];
}

// KB: k-values of the LDS images, 16 or 32; K <= KB.
template <int KIND, int KB>
__global__ void __launch_bounds__(256)
short_kernel(ShortArgs p)
{
    constexpr int PER = ST * KB / 256;  // elements per thread and operand
    constexpr int S = KIND == KIND_F32 ? 4 : kind_is_8bit(KIND) ? 1 : 2;
    __shared__ float As[KB][ST + 1], Bs[KB][ST + 1];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w >> 1, wn = w & 1;
    const int K = (int)p.K;
    const int64_t m0 = (int64_t)blockIdx.y * ST, n0 = (int64_t)blockIdx.x * ST, z = blockIdx.z;
    const char *A = p.A + (z * p.ms_a + (p.A_off ? p.A_off[0] : 0)) * S;
    const char *B = p.B + (z * p.ms_b + (p.B_off ? p.B_off[0] : 0)) * S;
    p.epi.C = (char *)p.epi.C + z * p.ms_c * (p.epi.c_f32 ? 4 : 2);

    // Threads run along the operand's contiguous direction.  Outside the matrix the nearest
    // element is read: nobody stores the rows and columns past the edge, and what lies past K
    // becomes zero in both operands (a zero in one would not undo an infinity in the other).
    const bool ak = p.transA == 0, bk = p.transB == 1 || p.b_packed;
    auto coord = [&](int e, bool k_fast, int &x, int &k) {
        const int i = e * 256 + tid;
        x = k_fast ? i / KB : i % ST;
        k = k_fast ? i % KB : i / ST;
    };
    float a[PER], b[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        int x, k;
        coord(e, ak, x, k);
        const int64_t m = m0 + x < p.M ? m0 + x : p.M - 1, at = k < K ? k : K - 1;
        a[e] = widen<KIND>(A, ak ? m * p.lda + at : at * p.lda + m);
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        int x, k;
        coord(e, bk, x, k);
        const int64_t n = n0 + x < p.N ? n0 + x : p.N - 1, at = k < K ? k : K - 1;
        b[e] = widen<KIND>(B, p.b_packed ? (at >> 3) * p.ldb + n * 8 + (at & 7) : bk ? n * p.ldb + at : at * p.ldb + n);
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        int x, k;
        coord(e, ak, x, k);
        As[k][x] = k < K ? a[e] : 0.0f;
        coord(e, bk, x, k);
        Bs[k][x] = k < K ? b[e] : 0.0f;
    }
    __syncthreads();

    // v_mfma_f32_32x32x2_f32: lane l supplies row l%32 of B^T and of A at k = l/32, and gets
    // row l%32 of C, four consecutive columns per group of four registers.
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        acc[r] = 0.0f;
    for (int k = 0; k < K; k += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Bs[k + (lane >> 5)][wn * 32 + (lane & 31)],
                                                   As[k + (lane >> 5)][wm * 32 + (lane & 31)], acc, 0, 0, 0);
    const int64_t m = m0 + wm * 32 + (lane & 31);
    if (m < p.M) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t n = n0 + wn * 32 + 8 * q + 4 * (lane >> 5);
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[i] = KIND == KIND_S8 ? __int_as_float((int)acc[4 * q + i]) : acc[4 * q + i];
            gen_store4(p.epi, m, n, p.N - n, v);
        }
    }
}

template <int KIND>
hipError_t launch_kind(const Problem &p)
{
    ShortArgs a;
    a.M = p.M; a.N = p.N; a.K = p.K; a.lda = p.lda; a.ldb = p.ldb;
    a.ms_a = p.ms_a; a.ms_b = p.ms_b; a.ms_c = p.ms_c;
    a.A = (const char *)p.A; a.B = (const char *)p.B;
    a.A_off = p.A_off; a.B_off = p.B_off;
    a.transA = p.transA; a.transB = p.transB; a.b_packed = p.b_packed;
    a.epi.beta = p.beta; a.epi.C = p.C; a.epi.ldc = p.ldc; a.epi.c_f32 = p.c_f32; a.epi.c_f16 = p.in_f16;
    a.epi.c_i32 = p.in_s8; a.epi.bias = p.bias; a.epi.relu = p.relu;
    const dim3 grid((unsigned)((p.N + ST - 1) / ST), (unsigned)((p.M + ST - 1) / ST), (unsigned)p.nmat);
    if (p.K <= 16)
        hipLaunchKernelGGL((short_kernel<KIND, 16>), grid, dim3(256), 0, p.stream, a);
    else
        hipLaunchKernelGGL((short_kernel<KIND, 32>), grid, dim3(256), 0, p.stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t general_launch_short(const Problem &p)
{
    if (p.batch != 1 || p.K > kMaxShort || p.split > 1)
        return hipErrorInvalidValue;
    if (p.in_s8)
        return launch_kind<KIND_S8>(p);
    if (p.in_f8)
        return p.f8_e5m2 ? launch_kind<KIND_BF8>(p) : launch_kind<KIND_F8>(p);
    if (p.in_f16)
        return launch_kind<KIND_F16>(p);
    return p.in_bf16 ? launch_kind<KIND_BF16>(p) : launch_kind<KIND_F32>(p);
}

}  // namespace brg
