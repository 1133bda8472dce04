// Elementwise passes: the sum of a reduction split's partial tiles with the epilogue, and
// the beta / bias / ReLU pass of a problem with an empty reduction.
#include "bf16_tiles.hpp"

namespace brg {

// Sum of the S partial results of an element in the order 0, 1, ..., S - 1.  S is a template
// argument so that all S loads are requested before the first is added: with a run-time loop the
// loads of a few slices at a time were waited for, and a short chain of latencies is all that
// bounds this kernel (bf16 16 x 4096 x 11008, 8 slices: the whole call 21.2 -> 20.1 us).
template <int S>
__global__ void __launch_bounds__(256)
reduce_kernel(int64_t M, int64_t N, const float *partial, Epilogue epi)
{
    const int64_t total = M * N;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        float v[S];
#pragma unroll
        for (int z = 0; z < S; ++z)
            v[z] = partial[(int64_t)z * total + e];
#pragma unroll
        for (int z = 1; z < S; ++z)
            v[0] += v[z];
        epilogue_store(epi, v[0], e / N, e % N);
    }
}

// The same sum, four consecutive columns per thread with 16-byte reads of the
// partial tiles (N a multiple of 4; C 16-byte aligned with ldc a multiple of 4).
template <int S>
__global__ void __launch_bounds__(256)
reduce4_kernel(int M, int quads_per_row, const float *partial, Epilogue epi)
{
    const int q = (int)blockIdx.x * 256 + (int)threadIdx.x;
    const int m = (int)blockIdx.y;
    if (q >= quads_per_row)
        return;
    const int64_t N = (int64_t)quads_per_row * 4;
    const int64_t total = (int64_t)M * N;
    const float *src = partial + (int64_t)m * N + (int64_t)q * 4;
    f32x4 v[S];
#pragma unroll
    for (int z = 0; z < S; ++z)
        v[z] = *(const f32x4 *)(src + (int64_t)z * total);
#pragma unroll
    for (int z = 1; z < S; ++z)
        v[0] += v[z];
    store4_epilogue(epi, m, (int64_t)q * 4, 4, true, v[0][0], v[0][1], v[0][2], v[0][3]);
}

__global__ void __launch_bounds__(256)
scale_only_kernel(int64_t M, int64_t N, Epilogue epi)
{
    const int64_t total = M * N;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256)
        epilogue_store(epi, 0.0f, e / N, e % N);
}

static Epilogue make_epilogue(const Problem &p)
{
    Epilogue e;
    e.beta = p.beta;
    e.C = p.C;
    e.ldc = p.ldc;
    e.c_f32 = p.c_f32;
    e.c_f16 = p.in_f16;
    e.c_i32 = p.in_s8;
    e.bias = p.bias;
    e.relu = p.relu;
    return e;
}

static unsigned elementwise_grid(int64_t total)
{
    int64_t g = (total + 255) / 256;
    if (g > 256 * 16)
        g = 256 * 16;
    if (g < 1)
        g = 1;
    return (unsigned)g;
}

template <int S>
static hipError_t launch_reduce_of(const Problem &p)
{
    if constexpr (S > kMaxSplit) {
        return hipErrorInvalidValue;
    } else {
        if (p.split != S)
            return launch_reduce_of<S + 1>(p);
        if ((p.N & 3) == 0 && (p.ldc & 3) == 0 && (((uintptr_t)p.C) & 15) == 0 && p.M <= 65535) {
            const int quads = (int)(p.N / 4);
            hipLaunchKernelGGL(reduce4_kernel<S>, dim3((unsigned)((quads + 255) / 256), (unsigned)p.M), dim3(256), 0,
                               p.stream, (int)p.M, quads, p.partial, make_epilogue(p));
        } else {
            hipLaunchKernelGGL(reduce_kernel<S>, dim3(elementwise_grid(p.M * p.N)), dim3(256), 0, p.stream, p.M, p.N,
                               p.partial, make_epilogue(p));
        }
        return hipGetLastError();
    }
}

hipError_t launch_reduce(const Problem &p) { return launch_reduce_of<2>(p); }

hipError_t launch_scale_only(const Problem &p)
{
    for (int64_t z = 0; z < p.nmat; ++z) {
        Epilogue e = make_epilogue(p);
        e.C = (char *)p.C + z * p.ms_c * (p.c_f32 ? 4 : 2);
        hipLaunchKernelGGL(scale_only_kernel, dim3(elementwise_grid(p.M * p.N)), dim3(256), 0, p.stream, p.M, p.N, e);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess)
            return err;
    }
    return hipSuccess;
}

}  // namespace brg
