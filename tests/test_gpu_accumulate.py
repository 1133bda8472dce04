"""Accumulating calls (fp32 C, beta != 0) whose old values and bias are requested ahead of the
epilogue: results at the tiles' edges, and that a bias costs no latency per store."""
import pytest
import torch

from paper_2511_13764_amd import binding as B

pytestmark = pytest.mark.gpu


def _ints(seed, *shape, lo=-3, hi=4):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(lo, hi, shape, device="cuda", generator=g, dtype=torch.int8).float()


def _call(dtype, M, N, K, A, W, beta, C, bias, **kw):
    code = {torch.float32: B.DTYPE_F32, torch.bfloat16: B.DTYPE_BF16, torch.float16: B.DTYPE_F16}[dtype]
    B.brgemm_fused(code, 0, 1, M, N, K, 1, A, None, K, W, None, K, beta, C, C.stride(0), 1, bias,
                   B.EPI_BIAS | B.EPI_RELU if bias is not None else 0, **kw)


# (M, N, K, form of the plan): whole and overhanging tiles of the kernels that read ahead
EDGES = [(torch.bfloat16, 81, 9176, 1024, "128x48"), (torch.float16, 128, 12284, 1088, "128x48"),
         (torch.bfloat16, 1500, 2044, 512, ""), (torch.float32, 1030, 1992, 96, ""), (torch.float32, 2048, 4100, 32, ""),
         (torch.bfloat16, 300, 328, 320, "32x32"), (torch.float32, 700, 1000, 64, "64x64"),
         (torch.bfloat16, 2001, 4004, 70, "128x128"), (torch.bfloat16, 1030, 2052, 70, "64x64")]


@pytest.mark.parametrize("dtype,M,N,K,form", EDGES)
@pytest.mark.parametrize("bias_shift", [None, 0, 1])
def test_old_values_and_bias_exact(dtype, M, N, K, form, bias_shift):
    """Integers below 2^24 in every sum: one result.  The bias starts on 16 bytes, off them, or is missing."""
    A, W = _ints(1, M, K).to(dtype), _ints(2, N, K).to(dtype)
    C0 = _ints(3, M, N, lo=-9, hi=10)
    bias = None if bias_shift is None else _ints(4, N + 1, lo=-9, hi=10)[bias_shift:bias_shift + N]
    ws = torch.empty(B.gemm_workspace_bytes(B.DTYPE_F32, M, N, K), dtype=torch.uint8, device="cuda")
    want = A.float().double() @ W.float().double().T + 2.0 * C0.double()
    if bias is not None:
        want = (want + bias.double()).clamp_min(0.0)
    for workspace in (ws, None):
        C = C0.clone()
        print(f"[gpu-case] {dtype} {M}x{N}x{K} {form} bias_shift={bias_shift} ws={workspace is not None}", flush=True)
        _call(dtype, M, N, K, A, W, 2.0, C, bias, workspace=workspace)
        if workspace is not None:
            assert B.gemm_form_name(B.gemm_last_form()) == form and B.gemm_last_split() == 1
        assert torch.equal(C.double(), want)


@pytest.mark.parametrize("dtype,M,N,K", [(torch.bfloat16, 2048, 2048, 256), (torch.float32, 2048, 2048, 64),
                                         (torch.bfloat16, 1000, 1000, 104)])
def test_a_bias_costs_little_beside_the_old_values(dtype, M, N, K):
    """Read between the stores the bias cost a latency each: 9.7 -> 12.9 us for the first of these."""
    A, W, C, bias = _ints(1, M, K).to(dtype), _ints(2, N, K).to(dtype), _ints(3, M, N), _ints(4, N)

    def us(b):
        for _ in range(20):
            _call(dtype, M, N, K, A, W, 1.0, C, b)
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = 1e9
        for _ in range(5):
            e[0].record()
            for _ in range(40):
                _call(dtype, M, N, K, A, W, 1.0, C, b)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) * 1e3 / 40)
        return best
    plain, with_bias = us(None), us(bias)
    print(f"[gpu-case] {dtype} {M}x{N}x{K}: {plain:.2f} us, with bias and ReLU {with_bias:.2f}", flush=True)
    assert with_bias <= 1.2 * plain
