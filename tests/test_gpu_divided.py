"""The general path's wide tiles, whose waves either load or multiply: against torch in 64 bits on
integer-valued operands (every sum below 2^24, so there is one result, to be met bit for bit)."""
import pytest
import torch

from paper_2511_13764_amd import binding as B

import gpu_helpers as H

pytestmark = pytest.mark.gpu

TYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32, "s8": torch.int8,
         "f8": torch.float8_e4m3fn, "bf8": torch.float8_e5m2}
CODE = {"bf16": B.DTYPE_BF16, "f16": B.DTYPE_F16, "f32": B.DTYPE_F32}
SUB = {"bf16": 64, "f16": 64, "f32": 32, "s8": 128, "f8": 64, "bf8": 64}
# (M, N, sub-blocks of k, k of the last one, first element, padding of the rows): tiles that end after one
# row or column, inside a chunk and on the tile's edge; the fewest steps, one turn of the register
# sets (3, 4, 5) and around it, whole and one-element K tails; rows on 2, 4 and 16 bytes
CASES = [(129, 65, 4, 1, 1, 0), (127, 200, 5, 0, 0, 0), (257, 130, 6, 63, 3, 1), (40, 333, 7, 8, 2, 6),
         (128, 256, 9, 0, 8, 8), (300, 71, 11, 31, 5, 3), (70, 130, 16, 5, 1, 1)]


def _operand(rows, cols, trans, shift, pad, dtype, gen):
    """Logical rows x cols small integers, and where they are stored: NaN (int8: 77) all around."""
    x = torch.randint(-2, 3, (rows, cols), generator=gen)
    st = x.T if trans else x
    ld = st.shape[1] + pad
    buf = torch.full((shift + st.shape[0] * ld + 16,), 77.0 if dtype == "s8" else float("nan")).to(TYPES[dtype])
    buf[shift:shift + st.shape[0] * ld].view(st.shape[0], ld)[:, :st.shape[1]] = st.to(TYPES[dtype])
    # the buffer ends with the last element a kernel may read
    end = shift + (st.shape[0] - 1) * ld + st.shape[1]
    return x, buf[:end].cuda()[shift:], ld


@pytest.mark.parametrize("dtype", list(TYPES))
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("form", ["128x128", "128x64", "64x64"])
def test_edges_tails_and_alignments_exact(dtype, tA, tB, form):
    gen = torch.Generator().manual_seed(29)
    form_id = next(f for f in range(8) if B.gemm_form_name(f) == form)
    for M, N, blocks, rest, shift, pad in CASES:
        K = SUB[dtype] * (blocks - 1) + (min(rest, SUB[dtype] - 1) or SUB[dtype])
        a, A, lda = _operand(M, K, tA, shift, pad, dtype, gen)
        w, W, ldb = _operand(K, N, tB, shift, pad, dtype, gen)
        c0 = torch.randint(-8, 9, (M, N), generator=gen)
        want = a @ w + c0
        ws = torch.empty(B.gemm_workspace_bytes(0, M, N, K), dtype=torch.uint8, device="cuda")
        C0 = c0.to(torch.int32 if dtype == "s8" else torch.float32).cuda()
        for split in (1, 2, 3) if dtype != "s8" else (1,):
            print(f"[gpu-case] {dtype} {form} t{tA}{tB} {M}x{N}x{K} shift={shift} pad={pad} split={split}", flush=True)
            C = C0.clone()
            B.gemm_force_variant(0, split)
            B.gemm_force_form(form_id)
            try:
                if dtype == "s8":
                    B.gemm_s8(tA, tB, M, N, K, A, lda, W, ldb, 1, C, N)
                elif dtype in CODE:
                    B.brgemm_fused(CODE[dtype], tA, tB, M, N, K, 1, A, None, lda, W, None, ldb, 1.0, C, N, 1, None, 0,
                                   workspace=ws)
                else:
                    (B.gemm_f8 if dtype == "f8" else B.gemm_bf8)(tA, tB, M, N, K, A, lda, W, ldb, 1.0, C, N, 1, workspace=ws)
            finally:
                B.gemm_force_variant(-1, 0)
            assert torch.equal(C.cpu().double(), want.double())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_two_workgroups_per_cu_and_batched_exact(dtype):
    """More tiles than CUs (the forms of four loading waves), and matrices of a batched call that start anywhere."""
    gen = torch.Generator().manual_seed(31)
    M, N, K, n = 271, 650, 5 * SUB[dtype] + 3, 9
    a, w = (torch.randint(-2, 3, s, generator=gen) for s in ((n, M, K), (n, K, N)))
    A, W = a.to(TYPES[dtype]).cuda(), w.to(TYPES[dtype]).cuda()
    want = a @ w
    for form in ("128x128", "128x64", "64x64"):
        C = torch.full((n, M, N), float("nan"), dtype=TYPES[dtype], device="cuda")
        print(f"[gpu-case] batched {dtype} {form}", flush=True)
        B.gemm_force_variant(0, 1)
        B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == form))
        try:
            if dtype == "bf16":
                B.gemm_bf16_batched(0, 0, M, N, K, n, A, K, M * K, W, N, K * N, 0.0, C, N, M * N, 0)
            else:
                B.gemm_f32_batched(0, 0, M, N, K, n, A, K, M * K, W, N, K * N, 0.0, C, N, M * N)
        finally:
            B.gemm_force_variant(-1, 0)
        assert torch.equal(C.cpu().double(), want.to(TYPES[dtype]).double())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("form", ["128x128", "128x64", "64x64"])
def test_long_sums_are_not_one_chain(dtype, form):
    """One product of 1 and K - 1 of which each instruction's sum is 0.9 of half an ulp of 1: one chain of fp32
    additions loses all of them, two chains half.  Closed off, only those beside the 1 are lost (at most an
    eighth here), and half an ulp at each of the K / 256 or more totals of 14 and more.  Sums past fp32's range are
    infinite, not NaN."""
    M, N, K = 130, 70, 8192
    per = 32 if dtype == "bf16" else 2          # products of one instruction
    a = torch.full((M, K + 1), 0.9 * 2.0 ** -24 / per, dtype=TYPES[dtype])          # (rows that no tuned kernel reads)
    small = float(a[0, 0]) * (K - 1)
    a[:, 0] = 1.0
    A, W, C = a.cuda(), torch.ones((N, K + 1), dtype=TYPES[dtype], device="cuda"), torch.empty((M, N), device="cuda")
    C_inf = torch.empty((M, N), device="cuda")
    A_inf = torch.full((M, K + 1), -3e38, dtype=TYPES[dtype], device="cuda")
    print(f"[gpu-case] long sums {dtype} {form}", flush=True)
    B.gemm_force_variant(0, 1)
    B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == form))
    try:
        for x, out in ((A, C), (A_inf, C_inf)):
            B.brgemm_fused(CODE[dtype], 0, 1, M, N, K, 1, x, None, K + 1, W, None, K + 1, 0.0, out, N, 1, None, 0)
            assert B.gemm_form_name(B.gemm_last_form()) == form and B.gemm_last_split() == 1
    finally:
        B.gemm_force_variant(-1, 0)
    off = (C.cpu().double() - (1.0 + small)).abs().max().item()
    assert off <= small / 4, (off, small)
    assert bool((C_inf == -float("inf")).all())


@pytest.mark.parametrize("form", ["128x128", "128x64", "64x64"])
@pytest.mark.parametrize("tA,K", [(0, 4 * 64 + 1), (1, 4 * 64 + 1), (0, 7 * 64 + 31), (1, 7 * 64 + 31)])
def test_packed_b_beside_rows_that_start_anywhere(form, tA, K):
    """B packed (its K padded with zeros), A's last sub-block incomplete and its rows off 16 bytes; bias, ReLU, and a C of
    either width whose rows start anywhere."""
    M, N = 333, 205
    gen = torch.Generator().manual_seed(61)
    a, A, lda = _operand(M, K, tA, 3, 1, "bf16", gen)
    w = torch.randint(-2, 3, (K, N), generator=gen)
    bias = torch.randint(-8, 9, (N,), generator=gen)
    W = w.to(torch.bfloat16).cuda()
    packed = torch.empty(B.gemm_packed_b_bytes(K, N) // 2, dtype=torch.bfloat16, device="cuda")
    B.gemm_pack_b_bf16(0, K, N, W, N, packed)
    want = (a @ w + bias).clamp_min(0).double()
    for c32, ldc, shift in ((1, N, 0), (1, N + 1, 1), (0, N + 1, 3), (0, N + 3, 0)):
        buf = torch.full((shift + M * ldc,), 99.0, dtype=torch.float32 if c32 else torch.bfloat16, device="cuda")
        C = buf[shift:].view(M, ldc)
        print(f"[gpu-case] packed {form} t{tA} K={K} c32={c32} ldc={ldc} shift={shift}", flush=True)
        B.gemm_force_variant(0, 1)
        B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == form))

        def call(stream=None):
            B.gemm_bf16_packed(tA, M, N, K, A, lda, packed, 0.0, buf[shift:], ldc, c32, dbias,
                               B.EPI_BIAS | B.EPI_RELU, stream=stream)
        dbias = bias.float().cuda()
        try:
            call()
            names = H.launched(call)
        finally:
            B.gemm_force_variant(-1, 0)
        assert len(names) == 1 and "general_duty_kernel" in names[0], names
        assert torch.equal(C[:, :N].cpu().double(), want if c32 else want.to(torch.bfloat16).double())
        assert bool((C[:, N:] == 99).all())


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("form", ["128x128", "128x64", "64x64"])
def test_bias_relu_and_unaligned_c_exact(dtype, form):
    M, N, K = 200, 141, 6 * SUB[dtype] + 5
    gen = torch.Generator().manual_seed(67)
    a, A, lda = _operand(M, K, 0, 1, 1, dtype, gen)
    w, W, ldb = _operand(K, N, 1, 1, 1, dtype, gen)
    c0, bias = torch.randint(-8, 9, (M, N), generator=gen), torch.randint(-8, 9, (N,), generator=gen)
    want = (a @ w + 2 * c0 + bias).clamp_min(0).double()
    dbias = bias.float().cuda()
    for c32, ldc, shift in ((1, N + 3, 0), (1, N + 1, 1)) + (((0, N + 1, 3),) if dtype != "f32" else ()):
        ct = torch.float32 if c32 else TYPES[dtype]
        buf = torch.full((shift + M * ldc,), 99.0, dtype=ct, device="cuda")
        C = buf[shift:].view(M, ldc)
        C[:, :N] = c0.to(ct).cuda()
        print(f"[gpu-case] fused {dtype} {form} c32={c32} ldc={ldc} shift={shift}", flush=True)
        B.gemm_force_variant(0, 1)
        B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == form))

        def call(stream=None):
            B.brgemm_fused(CODE[dtype], 0, 1, M, N, K, 1, A, None, lda, W, None, ldb, 2.0, buf[shift:], ldc, c32, dbias,
                           B.EPI_BIAS | B.EPI_RELU, stream=stream)
        try:
            call()
            names = H.launched(call)
        finally:
            B.gemm_force_variant(-1, 0)
        assert len(names) == 1 and "general_duty_kernel" in names[0], names
        assert torch.equal(C[:, :N].cpu().double(), want if c32 else want.to(ct).double())
        assert bool((C[:, N:] == 99).all())


# (type, layout, M, N, K, form, whether its waves are divided): either side of each line of the rule that says so
ROUTES = [("f32", 1, 1, 2228, 2534, 115, "128x128", False), ("f32", 1, 1, 2228, 2534, 384, "128x128", True),
          ("f32", 1, 1, 2000, 2000, 115, "128x128", True), ("f8", 0, 0, 2561, 830, 320, "128x64", False),
          ("f8", 0, 0, 1201, 830, 320, "128x64", True), ("f8", 0, 0, 2561, 830, 950, "128x64", True),
          ("f8", 0, 1, 2561, 830, 320, "128x64", True), ("f8", 0, 1, 4100, 1090, 320, "128x64", False),
          ("f8", 0, 1, 4100, 1090, 577, "128x64", True), ("f8", 1, 0, 4100, 1090, 1100, "128x64", False),
          ("s8", 0, 1, 463, 452, 579, "64x64", False), ("s8", 0, 1, 463, 452, 580, "64x64", True),
          ("s8", 0, 1, 463, 452, 1859, "64x64", True), ("s8", 0, 1, 463, 452, 579, "128x64", False),
          ("s8", 0, 1, 463, 452, 580, "128x64", True), ("s8", 1, 0, 463, 452, 640, "64x64", False),
          ("s8", 1, 0, 464, 448, 640, "64x64", True), ("s8", 1, 0, 463, 452, 640, "128x64", True),
          ("s8", 0, 0, 463, 452, 579, "64x64", True), ("s8", 0, 0, 2561, 830, 640, "128x64", False)]


@pytest.mark.parametrize("dtype,tA,tB,M,N,K,form,divided", ROUTES)
def test_which_products_are_divided(dtype, tA, tB, M, N, K, form, divided):
    gen = torch.Generator().manual_seed(53)
    a, A, lda = _operand(M, K, tA, 0, 0, dtype, gen)
    w, W, ldb = _operand(K, N, tB, 0, 0, dtype, gen)
    C = torch.full((M, N), 7 if dtype == "s8" else float("nan"), dtype=torch.int32 if dtype == "s8" else torch.float32, device="cuda")

    def call(stream=None):
        if dtype == "s8":
            B.gemm_s8(tA, tB, M, N, K, A, lda, W, ldb, 0, C, N, stream=stream)
        elif dtype == "f8":
            B.gemm_f8(tA, tB, M, N, K, A, lda, W, ldb, 0.0, C, N, 1, stream=stream)
        else:
            B.gemm_f32(tA, tB, M, N, K, A, lda, W, ldb, 0.0, C, N, stream=stream)
    print(f"[gpu-case] route {dtype} {form} t{tA}{tB} {M}x{N}x{K}", flush=True)
    B.gemm_force_variant(0, 1)
    B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == form))
    try:
        call()
        names = H.launched(call)
    finally:
        B.gemm_force_variant(-1, 0)
    assert torch.equal(C.cpu().double(), (a.float() @ w.float()).double())
    assert len(names) == 1 and ("general_duty_kernel" in names[0]) == divided, names


@pytest.mark.parametrize("dtype,tA,tB,M,N,K,form", [("f8", 1, 0, 1922, 1712, 383, "128x128"), ("f8", 0, 0, 928, 3440, 355, "128x128"),
                                                    ("s8", 1, 0, 1296, 3824, 7295, "128x128"), ("s8", 0, 0, 1344, 3744, 6979, "128x128"),
                                                    ("f8", 0, 1, 1000, 1001, 1500, "64x64"), ("s8", 0, 1, 1000, 1001, 1500, "64x64")])
def test_tiles_of_one_byte_products(dtype, tA, tB, M, N, K, form):
    """The plan's constants of the one-byte types are their own (the 16-bit ones prefer 128 x 64 in the first four)."""
    A, W = (torch.zeros(s, dtype=torch.int8, device="cuda") for s in ((K, M) if tA else (M, K), (N, K) if tB else (K, N)))
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    print(f"[gpu-case] plan {dtype} t{tA}{tB} {M}x{N}x{K}", flush=True)
    if dtype == "s8":
        B.gemm_s8(tA, tB, M, N, K, A, A.shape[1], W, W.shape[1], 0, C, N)
    else:
        B.gemm_f8(tA, tB, M, N, K, A, A.shape[1], W, W.shape[1], 0.0, C, N, 1)
    assert B.gemm_form_name(B.gemm_last_form()) == form
