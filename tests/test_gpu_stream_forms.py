"""The 64 x 64 and 128 x 64 tiles of 16-bit products whose rows global->LDS loads can read: against torch in 64 bits on
integer-valued operands (every sum below 2^24, so there is one result, to be met bit for bit)."""
import pytest
import torch

from paper_2511_13764_amd import binding as B

pytestmark = pytest.mark.gpu

TYPES = {"bf16": torch.bfloat16, "f16": torch.float16}
CODE = {"bf16": B.DTYPE_BF16, "f16": B.DTYPE_F16}
# (M, N, blocks of 64 k): one row or chunk past a tile, whole tiles, fewer blocks than the ring holds, as many, the
# blocks at which sums are closed off (4, 8) and one beside them, rows of C off 16 bytes
CASES = [(8, 8, 1), (72, 136, 2), (64, 64, 3), (136, 72, 4), (128, 200, 5), (264, 56, 8), (200, 328, 9), (65, 67, 6)]


def _forced(form, variant=0, split=1):
    B.gemm_force_variant(variant, split)
    B.gemm_force_form(next((f for f in range(8) if form and B.gemm_form_name(f) == form), -1))


@pytest.mark.parametrize("dtype", list(TYPES))
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("form", ["128x64", "64x64"])
def test_edges_splits_and_epilogues_exact(dtype, tA, tB, form):
    gen = torch.Generator().manual_seed(37)
    for M, N, blocks in CASES:
        K = 64 * blocks
        if (tA and M % 8) or (not tB and N % 8):
            continue
        a, w = (torch.randint(-2, 3, s, generator=gen) for s in ((M, K), (K, N)))
        bias = torch.randint(-8, 9, (N,), generator=gen)
        c0 = torch.randint(-8, 9, (M, N), generator=gen)
        A, W = ((x.T if t else x).contiguous().to(TYPES[dtype]).cuda() for x, t in ((a, tA), (w, tB)))
        ws = torch.empty(B.gemm_workspace_bytes(B.DTYPE_BF16, M, N, K), dtype=torch.uint8, device="cuda")
        want = (2 * c0 + a @ w + bias).clamp_min(0)
        for split in (1, 2, 3):
            for c32 in (0, 1):
                print(f"[gpu-case] {dtype} {form} t{tA}{tB} {M}x{N}x{K} split={split} c32={c32}", flush=True)
                C = c0.to(torch.float32 if c32 else TYPES[dtype]).cuda()
                _forced(form, 0, split)
                try:
                    B.brgemm_fused(CODE[dtype], tA, tB, M, N, K, 1, A, None, A.shape[1], W, None, W.shape[1], 2.0, C, N,
                                   c32, bias.float().cuda(), B.EPI_BIAS | B.EPI_RELU, workspace=ws)
                    assert B.gemm_form_name(B.gemm_last_form()) == form
                finally:
                    B.gemm_force_variant(-1, 0)
                assert torch.equal(C.cpu().double(), want.to(C.dtype).double())


@pytest.mark.parametrize("variant,M", [("bf16_stream_32x128x64", 33), ("bf16_stream_64x128x64", 65), ("bf16_stream_64x128x64", 300)])
@pytest.mark.parametrize("K", [512, 1280])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("form", ["", "64x64", "128x64"])
def test_the_streaming_variants_tiles_exact(variant, M, K, packed, form):
    """More rows than the variant's name and a long reduction: its full tiles, several below one another, and the tiles of as
    many elements that the automatic plan takes instead."""
    gen = torch.Generator().manual_seed(41)
    N = 200
    a, w = (torch.randint(-2, 3, s, generator=gen) for s in ((M, K), (K, N)))
    A, W = a.to(torch.bfloat16).cuda(), w.to(torch.bfloat16).cuda()
    C = torch.full((M, N), float("nan"), device="cuda")
    print(f"[gpu-case] {variant} {form} {M}x{N}x{K} packed={packed}", flush=True)
    _forced(form, B.variants().index(variant))
    try:
        if packed:
            image = torch.empty(B.gemm_packed_b_bytes(K, N) // 2, dtype=torch.bfloat16, device="cuda")
            B.gemm_pack_b_bf16(0, K, N, W, N, image)
            B.gemm_bf16_packed(0, M, N, K, A, K, image, 0.0, C, N, 1)
        else:
            B.gemm_bf16(0, 0, M, N, K, A, K, W, N, 0.0, C, N, 1)
        assert B.gemm_variant_name(B.gemm_last_variant()) == variant and B.gemm_form_name(B.gemm_last_form()) == form
    finally:
        B.gemm_force_variant(-1, 0)
    assert torch.equal(C.cpu().double(), (a @ w).double())


@pytest.mark.parametrize("variant,size,form", [("bf16_stream_32x128x64", 1024, "64x64"), ("bf16_stream_64x128x64", 1280, "128x64")])
def test_the_plan_reported_is_the_kernel_launched(variant, size, form):
    """Full tiles add a sum's terms as one chain, the tiles taken instead as two: the same bits say the same kernel."""
    A, W = (torch.randn((size, size), device="cuda", generator=torch.Generator("cuda").manual_seed(s)).to(torch.bfloat16) for s in (3, 4))

    def result(force):
        C = torch.full((size, size), float("nan"), device="cuda")
        if force is not None:
            _forced(force, B.variants().index(variant))
        try:
            B.gemm_bf16(0, 0, size, size, size, A, size, W, size, 0.0, C, size, 1)
            return C, B.gemm_variant_name(B.gemm_last_variant()), B.gemm_form_name(B.gemm_last_form())
        finally:
            B.gemm_force_variant(-1, 0)
    print(f"[gpu-case] kernels of {variant} at {size}", flush=True)
    auto, full, other = result(None), result(""), result(form)
    assert auto[1:] == other[1:] == (variant, form) and full[1:] == (variant, "")
    assert B.gemm_query_form(B.DTYPE_BF16, 0, 0, size, size, size) == form
    assert torch.equal(auto[0], other[0]) and not torch.equal(auto[0], full[0])


@pytest.mark.parametrize("form", ["128x64", "64x64"])
def test_batched_exact(form):
    gen = torch.Generator().manual_seed(43)
    n, M, N, K = 9, 136, 328, 320
    a, w = (torch.randint(-2, 3, s, generator=gen) for s in ((n, M, K), (n, K, N)))
    A, W = a.to(torch.bfloat16).cuda(), w.to(torch.bfloat16).cuda()
    C = torch.full((n, M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"[gpu-case] batched {form}", flush=True)
    _forced(form)
    try:
        B.gemm_bf16_batched(0, 0, M, N, K, n, A, K, M * K, W, N, K * N, 0.0, C, N, M * N, 0)
    finally:
        B.gemm_force_variant(-1, 0)
    assert torch.equal(C.cpu().double(), (a @ w).to(torch.bfloat16).double())


@pytest.mark.parametrize("M,N,K", [(1, 520, 65536), (40, 4096, 8256), (100, 16384, 2048), (130, 260, 131072)])
@pytest.mark.parametrize("split", [1, 3, 7])
def test_blocks_of_a_large_weight_matrix_taken_from_different_places(M, N, K, split):
    """Weights of 64 MB, rows along k: every streaming kernel that takes them, with slices of unequal length."""
    A = torch.randint(-2, 3, (M, K), device="cuda", generator=torch.Generator("cuda").manual_seed(47)).to(torch.bfloat16)
    W = torch.randint(-1, 2, (N, K), device="cuda", generator=torch.Generator("cuda").manual_seed(48)).to(torch.bfloat16)
    want = A.float() @ W.float().T              # (sums below 2^24 of integers: exact in any order)
    ws = torch.empty(split * M * N * 4, dtype=torch.uint8, device="cuda")
    for variant in ("bf16_stream_32x128x64", "bf16_stream_64x128x64", "bf16_stream_128x128x64"):
        C = torch.full((M, N), float("nan"), device="cuda")
        print(f"[gpu-case] rotated {variant} {M}x{N}x{K} split={split}", flush=True)
        _forced("", B.variants().index(variant), split)
        try:
            B.gemm_bf16(0, 1, M, N, K, A, K, W, K, 0.0, C, N, 1, workspace=ws)
        finally:
            B.gemm_force_variant(-1, 0)
        assert torch.equal(C, want)


def _large_weights(M, N, K, dtype, nmat=1):
    A = torch.randint(-2, 3, (nmat, M, K), device="cuda", generator=torch.Generator("cuda").manual_seed(61))
    W = torch.randint(-1, 2, (nmat, N, K), device="cuda", generator=torch.Generator("cuda").manual_seed(62))
    want = A.float() @ W.float().transpose(1, 2).contiguous()
    return *(x.to(torch.int8 if dtype == "s8" else torch.float32 if dtype == "f8" else torch.bfloat16) for x in (A, W)), want


@pytest.mark.parametrize("dtype", ["s8", "f8"])
@pytest.mark.parametrize("M,N,K", [(5, 1032, 65536), (200, 4104, 16512), (1000, 8100, 8320)])
def test_blocks_of_large_one_byte_weights_taken_from_different_places(dtype, M, N, K):
    """64 M elements and more: each streaming kernel that takes them, in slices of unequal length where they split."""
    A, W, want = _large_weights(M, N, K, dtype)
    A, W, want = A[0], W[0], want[0]
    if dtype == "f8":
        A, W = A.to(torch.float8_e4m3fn), W.to(torch.float8_e4m3fn)
    ws = torch.empty(3 * M * N * 4, dtype=torch.uint8, device="cuda")
    for variant in (None, "bf16_stream_32x128x64", "bf16_stream_64x128x64", "bf16_stream_128x128x64"):
        for split in (1, 3) if dtype == "f8" and variant else (1,):
            C = torch.full((M, N), -77, dtype=torch.int32 if dtype == "s8" else torch.float32, device="cuda")
            print(f"[gpu-case] rotated {dtype} {variant} {M}x{N}x{K} split={split}", flush=True)
            if variant:
                _forced("", B.variants().index(variant), split)
            try:
                if dtype == "s8":
                    B.gemm_s8(0, 1, M, N, K, A, K, W, K, 0, C, N)
                else:
                    B.gemm_f8(0, 1, M, N, K, A, K, W, K, 0.0, C, N, 1, workspace=ws)
            finally:
                B.gemm_force_variant(-1, 0)
            assert torch.equal(C.float(), want)


@pytest.mark.parametrize("M,N,K,variant", [(1000, 8100, 4160, "bf16_128x128x64"), (1, 4096, 8256, "bf16_stream_32x128x64"),
                                           (40, 8200, 4160, "bf16_stream_64x128x64"), (130, 4104, 8256, "bf16_stream_128x128x64")])
@pytest.mark.parametrize("nmat", [1, 2])
def test_blocks_of_large_weights_in_wide_tiles_and_batched_calls(M, N, K, variant, nmat):
    """(128 x 256 tiles are the two-stage variant's where one round of them covers C.)"""
    A, W, want = _large_weights(M, N, K, "bf16", nmat)
    C = torch.full((nmat, M, N), float("nan"), device="cuda")
    print(f"[gpu-case] rotated {variant} {M}x{N}x{K} x {nmat}", flush=True)
    _forced("", B.variants().index(variant), 1)
    try:
        B.gemm_bf16_batched(0, 1, M, N, K, nmat, A, K, M * K, W, K, N * K, 0.0, C, N, M * N, 1)
    finally:
        B.gemm_force_variant(-1, 0)
    assert torch.equal(C, want)


@pytest.mark.parametrize("M,tA,c32", [(768, 0, 0), (904, 1, 1)])
def test_without_allocation_as_with_a_workspace(M, tA, c32):
    """A plan whose partial sums exceed the library's buffer but took the place of one that needs none: same bits."""
    N, K = 4096, 8704
    gen = torch.Generator("cuda").manual_seed(53)
    A = torch.randn((K, M) if tA else (M, K), device="cuda", generator=gen).to(torch.bfloat16)
    W = torch.randn((N, K), device="cuda", generator=gen).to(torch.bfloat16)
    C = [torch.full((M, N), float("nan"), device="cuda").to(torch.float32 if c32 else torch.bfloat16) for _ in range(2)]
    ws = torch.empty(B.gemm_workspace_bytes(B.DTYPE_BF16, M, N, K), dtype=torch.uint8, device="cuda")
    print(f"[gpu-case] noalloc in rows of tiles {M}x{N}x{K} t{tA}1", flush=True)
    B.gemm_bf16(tA, 1, M, N, K, A, A.shape[1], W, K, 0.0, C[0], N, c32, workspace=ws)
    assert B.gemm_last_split() * M * N * 4 > B.NOALLOC_SCRATCH_BYTES
    B.gemm_bf16_noalloc(tA, 1, M, N, K, A, A.shape[1], W, K, 0.0, C[1], N, c32)
    torch.cuda.synchronize()
    assert torch.equal(C[0], C[1]) and not bool(C[0].isnan().any())


@pytest.mark.parametrize("variant", ["bf16_128x128x64", "bf16_pingpong_256x256x64", "bf16_stream_32x128x64",
                                     "bf16_stream_64x128x64", "bf16_stream_128x128x64"])
@pytest.mark.parametrize("at,ldc", [(0, 203), (1, 204), (2, 206), (3, 201)])
@pytest.mark.parametrize("c32,beta", [(0, 0.0), (0, 1.0), (1, 0.0), (1, 1.0)])
def test_rows_of_c_off_16_bytes_exact(variant, at, ldc, c32, beta):
    """Every column of every row, and nothing beside them: C starts `at` elements into its buffer, 201 columns of rows
    that start anywhere (the last group of four is incomplete)."""
    M, N, K = 131, 201, 192
    gen = torch.Generator().manual_seed(59)
    a, w = (torch.randint(-2, 3, s, generator=gen) for s in ((M, K), (K, N)))
    bias, c0 = torch.randint(-8, 9, (N,), generator=gen), torch.randint(-8, 9, (M, N), generator=gen)
    t = torch.float32 if c32 else torch.bfloat16
    A, W = a.to(torch.bfloat16).cuda(), w.T.contiguous().to(torch.bfloat16).cuda()
    buf = torch.full((at + M * ldc + 8,), 77.0, dtype=t, device="cuda")
    C = buf[at:at + M * ldc].view(M, ldc)
    C[:, :N] = c0.cuda().to(t) if beta else float("nan")
    ws = torch.empty(2 * M * N * 4, dtype=torch.uint8, device="cuda")
    for split in (1, 2):
        print(f"[gpu-case] odd C {variant} at={at} ldc={ldc} c32={c32} beta={beta} split={split}", flush=True)
        if beta:
            C[:, :N] = c0.cuda().to(t)
        _forced("", B.variants().index(variant), split)
        try:
            B.brgemm_fused(B.DTYPE_BF16, 0, 1, M, N, K, 1, A, None, K, W, None, K, beta, C, ldc, c32, bias.float().cuda(),
                           B.EPI_BIAS, workspace=ws)
        finally:
            B.gemm_force_variant(-1, 0)
        want = (a @ w + bias + (c0 if beta else 0)).double()
        assert torch.equal(C[:, :N].cpu().double(), want.to(t).double())
        assert bool((C[:, N:] == 77.0).all()) and bool((buf[:at] == 77.0).all()) and bool((buf[at + M * ldc:] == 77.0).all())
