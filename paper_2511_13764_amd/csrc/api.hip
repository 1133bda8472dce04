// Host side of the C ABI (include/brgemm.h): argument validation, choice of
// kernel variant and reduction split, launches on the caller's stream.
// The library never allocates, frees or synchronises.
#include "../../include/brgemm.h"
#include "common.hpp"
#include "variants.hpp"
#include <map>
#include <mutex>
#include <tuple>

using namespace brg;

// Library-owned partial-sum buffer of gemm_bf16_noalloc: device memory that is part of
// the code object, so no allocation call is ever made for it.  In host code this name
// is only a handle for hipGetSymbolAddress; the device address it yields (one per GPU)
// is what kernels and copies get.
constexpr size_t kScratchBytes = (size_t)BRGEMM_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

thread_local int tl_last_hip_error = 0;
thread_local int tl_forced_variant = -1;
thread_local int tl_forced_split = 0;
thread_local int tl_forced_form = -1;
thread_local int tl_last_variant = -1;
thread_local int tl_last_split = 0;
thread_local int tl_last_form = -1;

inline bool plan_is_forced() { return tl_forced_variant >= 0 || tl_forced_split > 0 || tl_forced_form >= 0; }
inline int forced_plan(const Problem &p, size_t workspace_bytes, Plan *out)
{
    return choose_plan(p, workspace_bytes, tl_forced_variant, tl_forced_split, tl_forced_form, out);
}
inline void remember(const Plan &plan)
{
    tl_last_variant = plan.variant;
    tl_last_split = plan.split;
    tl_last_form = plan.form;
}

inline int64_t stored_cols_a(const Problem &p) { return p.transA ? p.M : p.K; }
inline int64_t stored_cols_b(const Problem &p) { return p.transB ? p.K : p.N; }

constexpr int64_t kMaxDim = 2147483647LL;

inline int64_t round_up(int64_t x, int64_t to) { return (x + to - 1) / to * to; }

int validate(const Problem &p, const void *workspace, size_t workspace_bytes, bool need_offsets)
{
    if ((p.transA | 1) != 1 || (p.transB | 1) != 1)
        return BRGEMM_INVALID_ARG;
    if (p.M < 0 || p.N < 0 || p.K < 0 || p.batch < 0)
        return BRGEMM_INVALID_ARG;
    if (p.M > kMaxDim || p.N > kMaxDim || p.K > kMaxDim || p.batch > kMaxDim)
        return BRGEMM_INVALID_ARG;
    if (workspace_bytes > 0 && !workspace)
        return BRGEMM_INVALID_ARG;
    if (workspace && ((uintptr_t)workspace & 255u))
        return BRGEMM_MISALIGNED_WORKSPACE;
    if (p.M == 0 || p.N == 0)
        return BRGEMM_OK;
    if (!p.C || p.ldc < p.N)
        return BRGEMM_INVALID_ARG;
    if (p.K > 0 && p.batch > 0) {
        if (!p.A || !p.B)
            return BRGEMM_INVALID_ARG;
        if (p.lda < stored_cols_a(p) || p.ldb < stored_cols_b(p))
            return BRGEMM_INVALID_ARG;
        if (need_offsets && (!p.A_off || !p.B_off))
            return BRGEMM_INVALID_ARG;
        if ((p.A_off == nullptr) != (p.B_off == nullptr))
            return BRGEMM_INVALID_ARG;
        if (!p.A_off && p.batch > 1)
            return BRGEMM_INVALID_ARG;
    }
    return BRGEMM_OK;
}

int finish(hipError_t e)
{
    if (e != hipSuccess) {
        tl_last_hip_error = (int)e;
        return BRGEMM_HIP_ERROR;
    }
    return BRGEMM_OK;
}

// Device address of `scratch` on the current GPU, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_ptr[kMaxDevices] = {nullptr};

int scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices))
        e = hipErrorInvalidDevice;
    if (e == hipSuccess) {
        std::lock_guard<std::mutex> lock(scratch_mutex);
        if (!scratch_ptr[dev]) {
            void *ptr = nullptr;
            e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
            if (e == hipSuccess && !ptr)
                e = hipErrorInvalidSymbol;
            if (e == hipSuccess)
                scratch_ptr[dev] = ptr;
        }
        *out = scratch_ptr[dev];
    }
    if (e != hipSuccess) {
        tl_last_hip_error = (int)e;
        return BRGEMM_HIP_ERROR;
    }
    return BRGEMM_OK;
}

// Plans found by measurement (gemm_tune): shape -> (variant, split), consulted by every
// later call of the same element type, layout, sizes and leading dimensions.
typedef std::tuple<int, int, int, int, int, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t> TuneKey;
std::mutex tune_mutex;
std::map<TuneKey, Plan> tune_table;

TuneKey tune_key(const Problem &p)
{
    const int dtype = p.in_bf16 ? 1 : p.in_f16 ? 2 : p.in_s8 ? 3 : p.in_f8 ? (p.f8_e5m2 ? 5 : 4) : 0;
    return TuneKey(dtype, p.transA, p.transB, p.c_f32, p.b_packed, p.M, p.N, p.K, p.batch, p.lda, p.ldb);
}

bool tuned_plan(const Problem &p, size_t workspace_bytes, Plan *out)
{
    if (p.nmat != 1 || p.A_off)
        return false;
    Plan plan;
    {
        std::lock_guard<std::mutex> lock(tune_mutex);
        auto it = tune_table.find(tune_key(p));
        if (it == tune_table.end())
            return false;
        plan = it->second;
    }
    // the entry was measured on aligned operands with enough workspace: check this call's
    return choose_plan(p, workspace_bytes, plan.variant, plan.split, plan.form, out) == BRGEMM_OK;
}

// The plan of a call that forces and tunes nothing.
int automatic_plan(const Problem &p, size_t workspace_bytes, Plan *out)
{
    const int rc = choose_plan(p, workspace_bytes, -1, 0, -1, out);
    if (rc == BRGEMM_OK)
        prefer_small_tiles(p, workspace_bytes, out);
    return rc;
}

// Launch a planned problem.  HIP keeps the grid of a launch as 32-bit counts of threads and
// cuts a larger one off without an error (600,000,000 x 1 x 4 in 64 x 64 tiles of 512 threads
// returned success with 63 million rows written), so a C that could need 2^32 threads in the
// smallest tiles there are (32 x 32, 512 threads) is launched in halves.  They meet at a
// multiple of 256: a multiple of every tile and of every alignment rule.
hipError_t launch_planned(int variant, const Problem &p)
{
    const int64_t tiles = ((p.M + 31) / 32) * ((p.N + 31) / 32);
    if (tiles < ((int64_t)1 << 32) / 512) {
        hipError_t e = launch_variant(variant, p);
        if (e == hipSuccess && p.split > 1)
            e = launch_reduce(p);
        return e;
    }
    const int64_t esz = in_8bit(p) ? 1 : in_16bit(p) ? 2 : 4, csz = p.c_f32 ? 4 : 2;
    Problem half[2] = {p, p};
    Problem &q = half[1];
    if (p.M >= p.N) {
        const int64_t m = round_up(p.M / 2, 256);
        half[0].M = m;
        q.M = p.M - m;
        q.A = (const char *)p.A + m * (p.transA ? 1 : p.lda) * esz;
        q.C = (char *)p.C + m * p.ldc * csz;
    } else {
        const int64_t n = round_up(p.N / 2, 256);
        half[0].N = n;
        q.N = p.N - n;
        q.B = (const char *)p.B + n * (p.b_packed ? 8 : p.transB ? p.ldb : 1) * esz;
        q.C = (char *)p.C + n * csz;
        q.bias = p.bias ? p.bias + n : nullptr;
    }
    // (A split's partial tiles: the second half's replace the first half's on the stream.)
    const hipError_t e = launch_planned(variant, half[0]);
    return e == hipSuccess ? launch_planned(variant, q) : e;
}

// preset: a plan the caller has already chosen for this problem (nullptr: choose here).  library_scratch: the
// workspace is the library's own buffer, which is ordered between streams for split plans only; an unsplit
// launch gets no other workspace than its caller's.
int run(Problem &p, void *workspace, size_t workspace_bytes, bool need_offsets, const Plan *preset = nullptr,
        bool library_scratch = false)
{
    if (p.nmat == 0)
        p.nmat = 1;
    int rc = validate(p, workspace, workspace_bytes, need_offsets);
    if (rc != BRGEMM_OK)
        return rc;
    if (p.M == 0 || p.N == 0)
        return BRGEMM_OK;
    if (p.K == 0 || p.batch == 0) {
        if (p.beta == 1.0f && !p.bias && !p.relu)
            return BRGEMM_OK;               // C = 1*C: nothing to do
        remember(Plan{V_GENERIC, 1, -1});
        return finish(launch_scale_only(p));
    }

    Plan plan;
    if (preset)
        plan = *preset;
    else if (plan_is_forced())
        rc = forced_plan(p, workspace_bytes, &plan);
    else if (!tuned_plan(p, workspace_bytes, &plan))
        rc = automatic_plan(p, workspace_bytes, &plan);
    if (rc != BRGEMM_OK)
        return rc;
    p.split = plan.split;
    p.form = plan.form;
    p.partial = p.split > 1 ? (float *)workspace : nullptr;
    if (p.split == 1 && !library_scratch) {
        p.scratch = workspace;
        p.scratch_bytes = workspace_bytes;
    }

    const hipError_t e = launch_planned(plan.variant, p);
    if (e == hipSuccess)
        remember(plan);
    return finish(e);
}

}  // namespace

extern "C" {

int gemm_f32(int transA, int transB, int64_t M, int64_t N, int64_t K,
             const float *A, int64_t lda, const float *B, int64_t ldb,
             float beta, float *C, int64_t ldc,
             void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_bf16 = 0; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = 1;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_bf16(int transA, int transB, int64_t M, int64_t N, int64_t K,
              const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb,
              float beta, void *C, int64_t ldc, int c_is_f32,
              void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_bf16 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_bf16_noalloc(int transA, int transB, int64_t M, int64_t N, int64_t K,
                      const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb,
                      float beta, void *C, int64_t ldc, int c_is_f32, void *stream)
{
    Problem p{};
    p.in_bf16 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1; p.nmat = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    int rc = validate(p, nullptr, 0, false);
    if (rc != BRGEMM_OK)
        return rc;
    // The plan gemm_bf16 would take with all the workspace it can use must fit the
    // library's own buffer; a larger problem is refused, not run with another plan.
    Plan plan{V_GENERIC, 1, -1};
    const bool work = M > 0 && N > 0 && K > 0;
    int64_t rows = M;                               // of C, whose partial sums the buffer holds
    if (work) {
        rc = plan_is_forced() ? forced_plan(p, ~(size_t)0, &plan) : automatic_plan(p, ~(size_t)0, &plan);
        if (rc != BRGEMM_OK)
            return rc;
        const size_t slice = (size_t)M * (size_t)N * sizeof(float);
        // (a plan that took the place of one that fits, or needs no buffer: in rows of tiles, each of which does)
        const bool by_rows = plan.displaced > 0 && (plan.displaced == 1 || plan.displaced * slice <= kScratchBytes);
        rows = plan.split * slice <= kScratchBytes || plan.split == 1 ? M
               : by_rows ? (int64_t)(kScratchBytes / ((size_t)plan.split * (size_t)N * sizeof(float))) / 256 * 256 : 0;
        if (rows == 0)
            return BRGEMM_SCRATCH_TOO_SMALL;
    }
    void *ws = nullptr;
    rc = scratch_of_current_device(&ws);
    if (rc != BRGEMM_OK)
        return rc;
    if (rows < M) {
        // Whole tiles of 256 rows at a time, one after the other on the stream: the sums of a tile are the same.
        for (int64_t m = 0; m < M; m += rows) {
            Problem q = p;
            q.M = M - m < rows ? M - m : rows;
            q.A = (const uint16_t *)A + (transA ? m : m * lda);
            q.C = (char *)C + m * ldc * (p.c_f32 ? 4 : 2);
            rc = run(q, ws, kScratchBytes, false, &plan, true);
            if (rc != BRGEMM_OK)
                return rc;
        }
        return BRGEMM_OK;
    }
    return run(p, ws, kScratchBytes, false, work ? &plan : nullptr, true);
}

int gemm_f16(int transA, int transB, int64_t M, int64_t N, int64_t K,
             const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb,
             float beta, void *C, int64_t ldc, int c_is_f32,
             void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_f16 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_f8(int transA, int transB, int64_t M, int64_t N, int64_t K,
            const uint8_t *A, int64_t lda, const uint8_t *B, int64_t ldb,
            float beta, void *C, int64_t ldc, int c_is_f32,
            void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_f8 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_bf8(int transA, int transB, int64_t M, int64_t N, int64_t K,
             const uint8_t *A, int64_t lda, const uint8_t *B, int64_t ldb,
             float beta, void *C, int64_t ldc, int c_is_f32,
             void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_f8 = 1; p.f8_e5m2 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_s8(int transA, int transB, int64_t M, int64_t N, int64_t K,
            const int8_t *A, int64_t lda, const int8_t *B, int64_t ldb,
            int accumulate, int32_t *C, int64_t ldc, void *stream)
{
    Problem p{};
    p.in_s8 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = accumulate ? 1.0f : 0.0f; p.C = C; p.ldc = ldc; p.c_f32 = 1;
    p.stream = (hipStream_t)stream;
    return run(p, nullptr, 0, false);
}

int brgemm_bf16(int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t batch,
                const uint16_t *A_base, const int64_t *A_off, int64_t lda,
                const uint16_t *B_base, const int64_t *B_off, int64_t ldb,
                float beta, float *C, int64_t ldc,
                void *workspace, size_t workspace_bytes, void *stream)
{
    Problem p{};
    p.in_bf16 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = batch;
    p.A = A_base; p.A_off = A_off; p.lda = lda;
    p.B = B_base; p.B_off = B_off; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = 1;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, true);
}

int brgemm_fused(int in_dtype, int transA, int transB,
                 int64_t M, int64_t N, int64_t K, int64_t batch,
                 const void *A_base, const int64_t *A_off, int64_t lda,
                 const void *B_base, const int64_t *B_off, int64_t ldb,
                 float beta, void *C, int64_t ldc, int c_is_f32,
                 const float *bias, int epilogue,
                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (in_dtype != BRGEMM_DTYPE_F32 && in_dtype != BRGEMM_DTYPE_BF16 && in_dtype != BRGEMM_DTYPE_F16)
        return BRGEMM_INVALID_ARG;
    if (epilogue & ~(BRGEMM_EPI_BIAS | BRGEMM_EPI_RELU))
        return BRGEMM_INVALID_ARG;
    if ((epilogue & BRGEMM_EPI_BIAS) && !bias && N > 0)
        return BRGEMM_INVALID_ARG;
    if (in_dtype == BRGEMM_DTYPE_F32 && !c_is_f32)
        return BRGEMM_INVALID_ARG;
    Problem p{};
    p.in_bf16 = in_dtype == BRGEMM_DTYPE_BF16; p.in_f16 = in_dtype == BRGEMM_DTYPE_F16;
    p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = batch;
    p.A = A_base; p.A_off = A_off; p.lda = lda;
    p.B = B_base; p.B_off = B_off; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.bias = (epilogue & BRGEMM_EPI_BIAS) ? bias : nullptr;
    p.relu = (epilogue & BRGEMM_EPI_RELU) ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

int gemm_pack_vnni_bf16(int vnni, int transB, int64_t K, int64_t N, const uint16_t *B, int64_t ldb,
                        int64_t k_rows, int64_t n_pitch, uint16_t *out, void *stream)
{
    if ((transB | 1) != 1 || K < 0 || N < 0 || K > kMaxDim || N > kMaxDim)
        return BRGEMM_INVALID_ARG;
    if (vnni != 2 && vnni != 4 && vnni != 8)
        return BRGEMM_INVALID_ARG;
    if (k_rows < K || k_rows % vnni != 0 || n_pitch < N || k_rows > kMaxDim || n_pitch > kMaxDim)
        return BRGEMM_INVALID_ARG;
    if (k_rows == 0 || n_pitch == 0)
        return BRGEMM_OK;
    if (!out || ((uintptr_t)out & 15u))
        return BRGEMM_INVALID_ARG;
    if (K > 0 && N > 0 && (!B || ldb < (transB ? K : N)))
        return BRGEMM_INVALID_ARG;
    return finish(launch_pack_vnni(vnni, transB, K, N, B, ldb, k_rows, n_pitch, out, (hipStream_t)stream));
}

size_t gemm_packed_b_bytes(int64_t K, int64_t N)
{
    if (K <= 0 || N <= 0 || K > kMaxDim || N > kMaxDim)
        return 0;
    return (size_t)round_up(K, 64) * (size_t)round_up(N, 256) * sizeof(uint16_t);
}

int gemm_pack_b_bf16(int transB, int64_t K, int64_t N, const uint16_t *B, int64_t ldb,
                     uint16_t *packed, size_t packed_bytes, void *stream)
{
    if (K < 0 || N < 0 || K > kMaxDim || N > kMaxDim)
        return BRGEMM_INVALID_ARG;
    if (K == 0 || N == 0)
        return BRGEMM_OK;
    if (packed_bytes < gemm_packed_b_bytes(K, N))
        return BRGEMM_INVALID_ARG;
    return gemm_pack_vnni_bf16(8, transB, K, N, B, ldb, round_up(K, 64), round_up(N, 256), packed, stream);
}

int gemm_bf16_packed(int transA, int64_t M, int64_t N, int64_t K,
                     const uint16_t *A, int64_t lda, const uint16_t *packedB,
                     float beta, void *C, int64_t ldc, int c_is_f32,
                     const float *bias, int epilogue,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    if (epilogue & ~(BRGEMM_EPI_BIAS | BRGEMM_EPI_RELU))
        return BRGEMM_INVALID_ARG;
    if ((epilogue & BRGEMM_EPI_BIAS) && !bias && N > 0)
        return BRGEMM_INVALID_ARG;
    if (packedB && ((uintptr_t)packedB & 15u))
        return BRGEMM_INVALID_ARG;
    if (N > kMaxDim - 256)
        return BRGEMM_INVALID_ARG;
    Problem p{};
    p.in_bf16 = 1; p.transA = transA; p.transB = 0; p.b_packed = 1;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda;
    p.B = packedB; p.ldb = N > 0 ? round_up(N, 256) * 8 : 0;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.bias = (epilogue & BRGEMM_EPI_BIAS) ? bias : nullptr;
    p.relu = (epilogue & BRGEMM_EPI_RELU) ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run(p, workspace, workspace_bytes, false);
}

// Shared by the two batched entry points: the strides must describe matrices that fit
// (a stride of 0 shares an input operand; C matrices must not overlap).
static int run_batched(Problem &p, int64_t nmat, int64_t strideA, int64_t strideB, int64_t strideC)
{
    if (nmat < 0 || nmat > 65535 || strideA < 0 || strideB < 0 || strideC < 0)
        return BRGEMM_INVALID_ARG;
    if (nmat == 0)
        return BRGEMM_OK;
    if (nmat > 1 && p.M > 0 && p.N > 0 && strideC < (p.M - 1) * p.ldc + p.N)
        return BRGEMM_INVALID_ARG;
    p.nmat = nmat; p.ms_a = strideA; p.ms_b = strideB; p.ms_c = strideC;
    return run(p, nullptr, 0, false);
}

int gemm_bf16_batched(int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t nmat,
                      const uint16_t *A, int64_t lda, int64_t strideA,
                      const uint16_t *B, int64_t ldb, int64_t strideB,
                      float beta, void *C, int64_t ldc, int64_t strideC, int c_is_f32, void *stream)
{
    Problem p{};
    p.in_bf16 = 1; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    return run_batched(p, nmat, strideA, strideB, strideC);
}

int gemm_f32_batched(int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t nmat,
                     const float *A, int64_t lda, int64_t strideA,
                     const float *B, int64_t ldb, int64_t strideB,
                     float beta, float *C, int64_t ldc, int64_t strideC, void *stream)
{
    Problem p{};
    p.in_bf16 = 0; p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = beta; p.C = C; p.ldc = ldc; p.c_f32 = 1;
    p.stream = (hipStream_t)stream;
    return run_batched(p, nmat, strideA, strideB, strideC);
}

int gemm_tune(int dtype, int transA, int transB, int64_t M, int64_t N, int64_t K,
              const void *A, int64_t lda, const void *B, int64_t ldb,
              void *C, int64_t ldc, int c_is_f32,
              void *workspace, size_t workspace_bytes, void *stream,
              int *variant, int *split, float *microseconds)
{
    if (dtype != BRGEMM_DTYPE_F32 && dtype != BRGEMM_DTYPE_BF16 && dtype != BRGEMM_DTYPE_F16)
        return BRGEMM_INVALID_ARG;
    if (!variant || !split || M <= 0 || N <= 0 || K <= 0)
        return BRGEMM_INVALID_ARG;
    if (dtype == BRGEMM_DTYPE_F32 && !c_is_f32)
        return BRGEMM_INVALID_ARG;
    Problem p{};
    p.in_bf16 = dtype == BRGEMM_DTYPE_BF16; p.in_f16 = dtype == BRGEMM_DTYPE_F16;
    p.transA = transA; p.transB = transB;
    p.M = M; p.N = N; p.K = K; p.batch = 1; p.nmat = 1;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.beta = 0.0f; p.C = C; p.ldc = ldc; p.c_f32 = c_is_f32 ? 1 : 0;
    p.stream = (hipStream_t)stream;
    int rc = validate(p, workspace, workspace_bytes, false);
    if (rc != BRGEMM_OK)
        return rc;

    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t he = hipEventCreate(&e0);
    if (he == hipSuccess)
        he = hipEventCreate(&e1);
    Plan best{V_GENERIC, 1, -1};
    float best_us = -1.0f;
    static const int splits[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16};
    // The plan a call would take by itself first, then every variant and split; the general
    // kernel otherwise only when nothing else takes the problem.
    Plan candidates[1 + V_COUNT * (sizeof(splits) / sizeof(splits[0])) + 2];
    int count = automatic_plan(p, workspace_bytes, &candidates[0]) == BRGEMM_OK ? 1 : 0;
    bool tuned_kernel = false;
    for (int v = V_COUNT - 1; v >= 0; --v) {
        if (v == V_GENERIC && tuned_kernel)
            break;
        for (int s : splits) {
            if ((s == 1 || K / 64 / s >= 2) && choose_plan(p, workspace_bytes, v, s, -1, &candidates[count]) == BRGEMM_OK)
                ++count, tuned_kernel = tuned_kernel || v != V_GENERIC;
        }
    }
    for (int form : {(int)GEN_MID, (int)GEN_64}) {      // tiles that the automatic plan takes instead of full ones
        if (stream_form_runs(p, form) && choose_plan(p, workspace_bytes, V_GENERIC, 1, form, &candidates[count]) == BRGEMM_OK)
            ++count;
    }
    for (int c = 0; c < count; ++c) {
        const Plan &plan = candidates[c];
        // two untimed launches, then as many as fill about 300 us (at least 3)
        int reps = 3;
        for (int pass = 0; pass < 2 && he == hipSuccess; ++pass) {
            const int n = pass == 0 ? 2 : reps;
            he = hipEventRecord(e0, p.stream);
            for (int i = 0; i < n && he == hipSuccess; ++i) {
                Problem q = p;
                rc = run(q, workspace, workspace_bytes, false, &plan);
                if (rc != BRGEMM_OK)
                    he = hipErrorLaunchFailure;
            }
            if (he == hipSuccess)
                he = hipEventRecord(e1, p.stream);
            if (he == hipSuccess)
                he = hipEventSynchronize(e1);
            float ms = 0.0f;
            if (he == hipSuccess)
                he = hipEventElapsedTime(&ms, e0, e1);
            const float us = ms * 1000.0f / (float)n;
            if (pass == 0) {
                reps = us > 0.0f ? (int)(300.0f / us) : 3;
                reps = reps < 3 ? 3 : reps > 50 ? 50 : reps;
            } else if (he == hipSuccess && (best_us < 0.0f || us < best_us)) {
                best_us = us;
                best = plan;
            }
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (he != hipSuccess || best_us < 0.0f) {
        tl_last_hip_error = (int)he;
        return BRGEMM_HIP_ERROR;
    }
    {
        std::lock_guard<std::mutex> lock(tune_mutex);
        tune_table[tune_key(p)] = best;
    }
    remember(best);
    *variant = best.variant;
    *split = best.split;
    if (microseconds)
        *microseconds = best_us;
    return BRGEMM_OK;
}

void gemm_tune_reset(void)
{
    std::lock_guard<std::mutex> lock(tune_mutex);
    tune_table.clear();
}

size_t gemm_workspace_bytes(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch)
{
    (void)dtype;
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0)
        return 0;
    return (size_t)kMaxSplit * (size_t)M * (size_t)N * sizeof(float);
}

const char *gemm_strerror(int code)
{
    switch (code) {
    case BRGEMM_OK: return "success";
    case BRGEMM_INVALID_ARG: return "invalid argument (negative size, leading dimension too small, bad flag or NULL operand)";
    case BRGEMM_UNSUPPORTED: return "unsupported";
    case BRGEMM_WORKSPACE_TOO_SMALL: return "workspace too small for the forced split";
    case BRGEMM_HIP_ERROR: return "HIP launch error (see gemm_last_hip_error)";
    case BRGEMM_MISALIGNED_WORKSPACE: return "workspace is not 256-byte aligned";
    case BRGEMM_SCRATCH_TOO_SMALL: return "the problem's reduction split needs more than the library's built-in scratch buffer (gemm_bf16_noalloc)";
    default: return "unknown error code";
    }
}

int gemm_last_hip_error(void) { return tl_last_hip_error; }

int gemm_force_variant(int variant, int split)
{
    if (variant >= V_COUNT)
        return BRGEMM_INVALID_ARG;
    if (split > kMaxSplit)
        return BRGEMM_INVALID_ARG;
    tl_forced_variant = variant < 0 ? -1 : variant;
    tl_forced_split = split <= 0 ? 0 : split;
    tl_forced_form = -1;
    return BRGEMM_OK;
}

int gemm_force_form(int form)
{
    if (form >= 0 && !*form_name(form))
        return BRGEMM_INVALID_ARG;
    tl_forced_form = form < 0 ? -1 : form;
    return BRGEMM_OK;
}

static int query(int dtype, int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t batch,
                 int64_t lda, int64_t ldb, size_t workspace_bytes, Plan *plan)
{
    if (dtype != BRGEMM_DTYPE_F32 && dtype != BRGEMM_DTYPE_BF16 && dtype != BRGEMM_DTYPE_F16)
        return BRGEMM_INVALID_ARG;
    if ((transA | 1) != 1 || (transB | 1) != 1 || M <= 0 || N <= 0 || K <= 0 || batch <= 0)
        return BRGEMM_INVALID_ARG;
    Problem p{};
    p.in_bf16 = dtype == BRGEMM_DTYPE_BF16; p.in_f16 = dtype == BRGEMM_DTYPE_F16;
    p.transA = transA; p.transB = transB; p.M = M; p.N = N; p.K = K; p.batch = batch; p.nmat = 1;
    // stand-ins for 16-byte aligned operands (never dereferenced); batch > 1 means tile offsets
    p.A = (const void *)0x1000; p.B = (const void *)0x1000; p.C = (void *)0x1000;
    p.A_off = batch > 1 ? (const int64_t *)0x1000 : nullptr; p.B_off = p.A_off;
    p.lda = lda; p.ldb = ldb; p.ldc = N; p.c_f32 = 1;
    if (p.lda < stored_cols_a(p) || p.ldb < stored_cols_b(p))
        return BRGEMM_INVALID_ARG;
    return automatic_plan(p, workspace_bytes, plan);
}

int gemm_query_plan(int dtype, int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t batch,
                    int64_t lda, int64_t ldb, size_t workspace_bytes, int *variant, int *split)
{
    Plan plan;
    if (!variant || !split)
        return BRGEMM_INVALID_ARG;
    const int rc = query(dtype, transA, transB, M, N, K, batch, lda, ldb, workspace_bytes, &plan);
    if (rc != BRGEMM_OK)
        return rc;
    *variant = plan.variant;
    *split = plan.split;
    return BRGEMM_OK;
}

int gemm_query_form(int dtype, int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t batch,
                    int64_t lda, int64_t ldb, size_t workspace_bytes, int *form)
{
    Plan plan;
    if (!form)
        return BRGEMM_INVALID_ARG;
    const int rc = query(dtype, transA, transB, M, N, K, batch, lda, ldb, workspace_bytes, &plan);
    if (rc != BRGEMM_OK)
        return rc;
    *form = plan.form;
    return BRGEMM_OK;
}

const char *gemm_variant_name(int v) { return variant_name(v); }
int gemm_last_variant(void) { return tl_last_variant; }
int gemm_last_split(void) { return tl_last_split; }
const char *gemm_form_name(int form) { return form_name(form); }
int gemm_last_form(void) { return tl_last_form; }

}  // extern "C"
