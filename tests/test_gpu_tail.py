"""16-bit problems whose K ends inside a block of 64 on the tuned kernels' tiles (the general path's
128 x 128 form routes them): integer operands, so one result, to be met bit for bit."""
import pytest
import torch

from paper_2511_13764_amd import binding as B

import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _stored(x, trans, dtype):
    """x as a program stores it, rows on 16 bytes, NaN in the padding; the buffer ends with the last element."""
    st = x.T if trans else x
    ld = (st.shape[1] + 7) // 8 * 8
    buf = torch.full((st.shape[0] * ld,), float("nan"), dtype=dtype)
    buf.view(st.shape[0], ld)[:, :st.shape[1]] = st.to(dtype)
    return buf[:(st.shape[0] - 1) * ld + st.shape[1]].cuda(), ld


# one tile row / column more than whole tiles, the grids of each kernel: up to 256 tiles of 128 x 128 (whole
# and split), up to 256 of 128 x 256, more (general tiles at this K); the 48-column weight stream (NT only)
SHAPES = [(264, 136, (1, 2, 3)), (2312, 2184, (1,)), (2952, 3208, (1,)), (104, 9608, (1,))]


def _tile(M, N, weights):
    """Kernel and, of the streaming kernel's tiles, columns that a shape above is meant for (`weights`: both operands along k)."""
    if (M, N) == (104, 9608) and weights:
        return "bf16_stream128_kernel", "Li48ELb1E"
    tiles, wide = -(-M // 128) * -(-N // 128), -(-M // 128) * -(-N // 256)
    return ("bf16_stream128_kernel", "Li128ELb1E") if tiles <= 256 else ("bf16_stream128_kernel", "Li256ELb1E") if wide <= 256 else ("general_kernel", "")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,splits", SHAPES)
@pytest.mark.parametrize("K", [513, 575, 600])
def test_incomplete_last_block_exact(dtype, tA, tB, M, N, splits, K):
    _exact(dtype, tA, tB, M, N, splits, K, _tile(M, N, tA == 0 and tB == 1))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K", [961, 1000, 1023])
def test_incomplete_last_block_of_256_tiles_exact(dtype, tA, tB, K):
    _exact(dtype, tA, tB, 3848, 3592, (1,), K, ("bf16_pingpong_kernel",))


def _exact(dtype, tA, tB, M, N, splits, K, kernel):
    gen = torch.Generator().manual_seed(37)
    a, w = (torch.randint(-2, 3, s, generator=gen).float() for s in ((M, K), (K, N)))
    want = a @ w
    A, lda = _stored(a, tA, dtype)
    W, ldb = _stored(w, tB, dtype)
    call = B.gemm_bf16 if dtype == torch.bfloat16 else B.gemm_f16
    form = next(f for f in range(8) if B.gemm_form_name(f) == "128x128")
    ws = torch.empty(B.gemm_workspace_bytes(0, M, N, K), dtype=torch.uint8, device="cuda")
    for split in splits:
        print(f"[gpu-case] {dtype} t{tA}{tB} {M}x{N}x{K} split={split}", flush=True)
        C = torch.full((M, N), 2.0, device="cuda")
        B.gemm_force_variant(0, split)
        B.gemm_force_form(form)
        try:
            call(tA, tB, M, N, K, A, lda, W, ldb, 1.0, C, N, 1, workspace=ws)
            names = H.launched(lambda s: call(tA, tB, M, N, K, A, lda, W, ldb, 1.0, C, N, 1, workspace=ws, stream=s))
        finally:
            B.gemm_force_variant(-1, 0)
        assert torch.equal(C.cpu(), want + 2.0)
        assert len(names) == (2 if split > 1 else 1) and all(part in names[0] for part in kernel), names


# (rows of C off 16 bytes: the 256 x 256 kernel's rounds do not pay for 2952 x 3205; 3208 columns do)
KERNEL_OF_PACKED = {(264, 130): "Li128ELb1E", (2312, 2181): "Li256ELb1E", (2952, 3205): "general_kernel", (2952, 3208): "bf16_pingpong_kernel"}


@pytest.mark.parametrize("tA", [0, 1])
@pytest.mark.parametrize("M,N", list(KERNEL_OF_PACKED))
def test_packed_b_and_16_bit_c(tA, M, N):
    K = 1000
    gen = torch.Generator().manual_seed(41)
    a, w = (torch.randint(-1, 2, s, generator=gen).float() for s in ((M, K), (K, N)))
    A, lda = _stored(a, tA, torch.bfloat16)
    W = w.to(torch.bfloat16).cuda()
    packed = torch.empty(B.gemm_packed_b_bytes(K, N) // 2, dtype=torch.bfloat16, device="cuda")
    B.gemm_pack_b_bf16(0, K, N, W, N, packed)
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"[gpu-case] packed tA={tA} {M}x{N}", flush=True)
    B.gemm_force_variant(0, 1)
    B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == "128x128"))
    try:
        B.gemm_bf16_packed(tA, M, N, K, A, lda, packed, 0.0, C, N, 0)
        names = H.launched(lambda s: B.gemm_bf16_packed(tA, M, N, K, A, lda, packed, 0.0, C, N, 0, stream=s))
    finally:
        B.gemm_force_variant(-1, 0)
    assert torch.equal(C.cpu(), (a @ w).to(torch.bfloat16))
    assert len(names) == 1 and (KERNEL_OF_PACKED[(M, N)] in names[0]), names


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K,shift,pad", [(2305, 1, 0), (2304, 0, 1), (2311, 3, 2), (2304, 8, 8)])
def test_rows_copied_into_the_workspace_exact(tA, tB, K, shift, pad):
    """Large problems whose rows start anywhere: operands that need it are copied, with a workspace that holds
    them, else nothing is; the same result, and nothing behind the copies is written."""
    M, N = 3849, 3841
    gen = torch.Generator(device="cuda").manual_seed(43)
    a, w = (torch.randint(-2, 3, s, generator=gen, device="cuda").float() for s in ((M, K), (K, N)))
    want = a @ w + 3.0                          # integers below 2^24: exact in any order

    def stored(x, trans):
        st = x.T if trans else x
        ld = st.shape[1] + pad
        buf = torch.full((shift + st.shape[0] * ld,), float("nan"), dtype=torch.bfloat16, device="cuda")
        buf[shift:].view(st.shape[0], ld)[:, :st.shape[1]] = st.to(torch.bfloat16)
        return buf[shift:shift + (st.shape[0] - 1) * ld + st.shape[1]], ld
    (A, lda), (W, ldb) = stored(a, tA), stored(w, tB)
    need = sum((r * ((c + 63) // 64 * 64) * 2 + 255) // 256 * 256
               for (r, c), mn in (((K, M) if tA else (M, K), tA), ((N, K) if tB else (K, N), not tB))
               if shift % 8 or (c + pad) % 8 or (mn and c % 8))
    for size in (need + 4096, need - 256, 0):
        ws = torch.full((max(size, 0),), 0x5A, dtype=torch.uint8, device="cuda") if size > 0 else None
        print(f"[gpu-case] realigned t{tA}{tB} {M}x{N}x{K} shift={shift} pad={pad} workspace={size}", flush=True)
        C = torch.full((M, N), 3.0, device="cuda")
        B.gemm_bf16(tA, tB, M, N, K, A, lda, W, ldb, 1.0, C, N, 1, workspace=ws)
        assert torch.equal(C, want)
        if ws is not None and size > need > 0 and B.gemm_last_split() == 1:
            assert bool((ws[need:] == 0x5A).all())
            assert not bool((ws[:need] == 0x5A).all())


@pytest.mark.parametrize("M,N", [(264, 136), (104, 9608)])
def test_long_sums_are_not_one_chain(M, N):
    """One product of 1 and K - 1 of which each instruction's sum (32 products) is 0.9 of half an ulp of 1: one chain
    of fp32 additions loses all of them, totals every 16 blocks of 64 lose an eighth."""
    K = 8200
    a = torch.full((M, K), 0.9 * 2.0 ** -29, dtype=torch.bfloat16)
    small = float(a[0, 0]) * (K - 1)
    a[:, 0] = 1.0
    C = torch.empty((M, N), device="cuda")
    print(f"[gpu-case] long sums {M}x{N}x{K}", flush=True)
    B.gemm_force_variant(0, 1)
    B.gemm_force_form(next(f for f in range(8) if B.gemm_form_name(f) == "128x128"))
    try:
        A, W = a.cuda(), torch.ones((N, K), dtype=torch.bfloat16, device="cuda")
        B.gemm_bf16(0, 1, M, N, K, A, K, W, K, 0.0, C, N, 1)
        names = H.launched(lambda s: B.gemm_bf16(0, 1, M, N, K, A, K, W, K, 0.0, C, N, 1, stream=s))
    finally:
        B.gemm_force_variant(-1, 0)
    assert (C.cpu().double() - (1.0 + small)).abs().max().item() <= small / 4
    assert len(names) == 1 and all(part in names[0] for part in _tile(M, N, True)), names


# (A^T, B^T, M, N, K, rows on 16 bytes, the kernels of the call): more than 512 tiles of 128 x 128, whose 256 x 256 tiles
# fill the chip's rounds or begin another with a few
PP, COPY, GENERAL = "bf16_pingpong_kernel", "realign_kernel", "general_kernel"
ROUTES = [(0, 1, 4096, 4096, 1000, True, [PP]), (1, 1, 2384, 6728, 835, True, [GENERAL]), (0, 0, 2648, 7160, 528, True, [GENERAL]),
          (0, 1, 3840, 3841, 840, True, [GENERAL]), (0, 1, 3840, 3844, 840, True, [PP]),
          (0, 1, 4096, 4096, 2305, False, [COPY, PP]), (1, 0, 3849, 3841, 2304, False, [COPY, PP]),
          (0, 0, 1503, 9730, 625, False, [GENERAL]), (1, 1, 1371, 9678, 705, False, [GENERAL])]


@pytest.mark.parametrize("tA,tB,M,N,K,rows16,kernels", ROUTES)
def test_rounds_decide_between_the_tiles(tA, tB, M, N, K, rows16, kernels):
    gen = torch.Generator(device="cuda").manual_seed(59)

    def operand(rows, cols, trans):
        x = torch.randint(-2, 3, (rows, cols), generator=gen, device="cuda").float()
        if rows16:
            return x, *_stored(x, trans, torch.bfloat16)
        st = (x.T if trans else x).to(torch.bfloat16).contiguous()
        return x, st, st.shape[1]
    (a, A, lda), (w, W, ldb) = operand(M, K, tA), operand(K, N, tB)
    C = torch.empty((M, N), device="cuda")
    ws = torch.empty(4 * (M + N) * (K + 64), dtype=torch.uint8, device="cuda")          # the copies, not partial sums
    print(f"[gpu-case] route t{tA}{tB} {M}x{N}x{K} rows16={rows16}", flush=True)

    def call(stream=None):
        B.gemm_bf16(tA, tB, M, N, K, A, lda, W, ldb, 0.0, C, N, 1, workspace=ws, stream=stream)
    call()
    assert torch.equal(C, a @ w)                # integers below 2^24: exact in any order
    names = H.launched(call)
    assert len(names) == len(kernels) and all(k in n for k, n in zip(kernels, names)), names
