"""The calls whose time this framework is judged by, and what their results have to be.

Each case is one call of a public entry point as a program makes it: operands, weights,
outputs and a workspace already on the GPU, one library call per pass.  Sizes are those of
the repository's own workloads (fp32 squares, bf16 squares, transformer-MLP layers with
4096 x 11008 weights, batch-reduce over scattered tiles) or generic ones around them;
`draw` spreads the same kinds of call over their whole range, odd sizes among them.
"""
import math

import torch

from paper_2511_13764_amd import binding as B

GEMM_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16,
               "s8": torch.int8, "f8": torch.float8_e4m3fn, "bf8": torch.float8_e5m2}
WORKSPACE_CAP = 1 << 30
MAX_FLOPS = 2.0 * 4096 * 11008 * 4096          # of a drawn case: the largest listed one's
POOL_TILE_ALIGN = 64                           # elements; tiles of a batch-reduce call start on 128 bytes


def _gemm(name, dtype, tA, tB, M, N, K, beta=0.0, c32=False, pad=0, bias=False, relu=False, packed=False):
    return {"name": name, "kind": "gemm", "dtype": dtype, "tA": tA, "tB": tB, "M": M, "N": N, "K": K,
            "beta": beta, "c32": bool(c32 or dtype == "f32"), "pad": pad, "bias": bias, "relu": relu, "packed": packed}


def listed():
    return [
        # the smallest fp32 product of the workloads: launch and latency
        _gemm("f32_256", "f32", 0, 0, 256, 256, 256),
        # fp32 with an accumulating C at the size where the matrix units set the time
        _gemm("f32_2048_beta", "f32", 0, 0, 2048, 2048, 2048, beta=0.5),
        # fp32 on sizes that are a multiple of nothing, second operand transposed (a least-squares
        # or covariance product of data as it comes)
        _gemm("f32_odd", "f32", 0, 1, 777, 1001, 1301),
        # small and headline squares of the bf16 sweep
        _gemm("bf16_1024", "bf16", 0, 0, 1024, 1024, 1024),
        _gemm("bf16_4096", "bf16", 0, 0, 4096, 4096, 4096),
        # bf16 layer whose sequence length and widths are not multiples of the tiles
        _gemm("bf16_odd", "bf16", 0, 1, 1000, 2003, 1500),
        # prefill through an MLP layer with its bias and ReLU; weights stored N x K
        _gemm("mlp_up_4096_bias_relu", "bf16", 0, 1, 4096, 11008, 4096, bias=True, relu=True),
        # the same weights for a batch of 128 and for the decode of 16 sequences
        _gemm("mlp_up_128", "bf16", 0, 1, 128, 11008, 4096),
        _gemm("mlp_down_16", "bf16", 0, 1, 16, 4096, 11008),
        # weight gradient of the down-projection over 1024 tokens, accumulated in fp32
        _gemm("grad_down_1024", "bf16", 1, 0, 4096, 11008, 1024, beta=1.0, c32=True),
        # batch-reduce over tiles scattered in a pool
        {"name": "brgemm_scattered", "kind": "brgemm", "M": 512, "N": 512, "K": 64, "batch": 64, "beta": 1.0},
        # one-byte operands
        _gemm("f8_4096", "f8", 0, 1, 4096, 4096, 4096),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size of the range: as it falls, or rounded to what programs like (multiples of 64, of 8)."""
    x = _logint(rng, lo, hi)
    how = rng.random()
    if how < 0.5:
        return max(64, (x + 32) // 64 * 64) if hi >= 64 else x
    if how < 0.7:
        return max(8, (x + 4) // 8 * 8)
    return x


def draw(rng):
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= MAX_FLOPS:
            return c


def _draw(rng):
    kind = rng.choices(["f32", "square", "mlp", "grad", "brgemm", "batched", "bytes"], [3, 4, 5, 2, 2, 2, 2])[0]
    tA, tB = rng.choice([(0, 0), (0, 0), (0, 1), (0, 1), (1, 0), (1, 1)])
    if kind == "f32":
        c = _gemm("", "f32", tA, tB, _size(rng, 64, 2048), _size(rng, 64, 2048), _size(rng, 64, 2048),
                  beta=rng.choice([0.0, 0.0, 0.5, 1.0]), pad=rng.choice([0, 0, 0, 8]))
    elif kind == "square":
        c = _gemm("", rng.choice(["bf16", "bf16", "f16"]), tA, tB, _size(rng, 128, 4096), _size(rng, 128, 4096),
                  _size(rng, 128, 4096), c32=rng.random() < 0.25, pad=rng.choice([0, 0, 0, 8]))
    elif kind == "mlp":
        M = _logint(rng, 1, 4096)
        if M > 64 and rng.random() < 0.5:
            M = (M + 63) // 64 * 64
        K, N = rng.choice([(4096, 11008), (11008, 4096), (4096, 4096),
                           (_size(rng, 512, 8192), _size(rng, 512, 8192))])
        act = rng.random() < 0.5
        c = _gemm("", "bf16", 0, 1, M, N, K, bias=act, relu=act, packed=rng.random() < 0.25)
    elif kind == "grad":
        # weight gradient (A transposed, fp32 sums) or input gradient (plain) of a layer
        T, K, N = _size(rng, 128, 4096), _size(rng, 512, 4096), _size(rng, 512, 4096)
        c = (_gemm("", "bf16", 1, 0, K, N, T, beta=1.0, c32=True) if rng.random() < 0.6
             else _gemm("", "bf16", 0, 0, T, N, K))
    elif kind == "brgemm":
        c = {"kind": "brgemm", "M": _size(rng, 32, 1024), "N": _size(rng, 64, 1024),
             "K": rng.choice([32, 64, 64, 128, 256, _logint(rng, 17, 250)]), "batch": _logint(rng, 4, 96),
             "beta": rng.choice([0.0, 1.0])}
    elif kind == "batched":
        c = {"kind": "batched", "dtype": rng.choice(["bf16", "f32"]), "tA": tA, "tB": tB, "M": _size(rng, 32, 512),
             "N": _size(rng, 32, 512), "K": _size(rng, 32, 512), "nmat": _logint(rng, 4, 64),
             "beta": rng.choice([0.0, 0.0, 1.0])}
    else:
        c = _gemm("", rng.choice(["s8", "f8", "bf8"]), tA, tB, _size(rng, 16, 4096), _size(rng, 256, 4096),
                  _size(rng, 256, 4096))
        if c["dtype"] == "s8":
            c["c32"] = True
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs

def _values(shape, dtype, gen, weights=False):
    """Stored operand: uniform[-1, 1] in fp32, N(0, 1) activations and N(0, 0.02) weights in the
    narrow types (one-byte floats N(0, 1): their weights carry a scale), all codes in int8."""
    if dtype == "s8":
        return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=gen)
    if dtype == "f32":
        return torch.rand(shape, device="cuda", generator=gen) * 2.0 - 1.0
    x = torch.randn(shape, device="cuda", generator=gen)
    if weights and dtype in ("bf16", "f16"):
        x *= 0.02
    return x.to(GEMM_DTYPES[dtype])


def _stored(rows, cols, trans, pad, dtype, gen, weights=False):
    r, c = (cols, rows) if trans else (rows, cols)
    return _values((r, c + pad), dtype, gen, weights)


def _out_dtype(case):
    if case["dtype"] == "s8":
        return torch.int32
    if case["c32"]:
        return torch.float32
    return torch.float16 if case["dtype"] == "f16" else torch.bfloat16


def _tiles(case, gen):
    """Pool and tile offsets of a batch-reduce call: tiles at random places, not in order."""
    M, N, K, n = case["M"], case["N"], case["K"], case["batch"]
    slot = (max(M * K, K * N) + 2 * POOL_TILE_ALIGN) // POOL_TILE_ALIGN * POOL_TILE_ALIGN
    slots = max(2 * n, (32 << 20) // slot)                   # a 64 MiB pool where the tiles fit one
    pool = torch.full((slots * slot,), float("nan"), dtype=torch.bfloat16, device="cuda")
    order = torch.randperm(slots, device="cuda", generator=gen)[:2 * n]
    starts = order * slot
    rows = torch.arange(max(M * K, K * N), device="cuda")
    for first, size in ((0, M * K), (n, K * N)):
        at = (starts[first:first + n, None] + rows[None, :size]).reshape(-1)
        pool[at] = _values((n * size,), "bf16", gen)
    return pool, starts[:n].clone(), starts[n:].clone()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    M, N, K = case["M"], case["N"], case["K"]
    s = {"case": case}
    if case["kind"] == "brgemm":
        s["pool"], s["A_off"], s["B_off"] = _tiles(case, gen)
        s["C"] = torch.randn((M, N), device="cuda", generator=gen)
        s["ws"] = _workspace(B.DTYPE_BF16, M, N, K, case["batch"])
    elif case["kind"] == "batched":
        n, dt = case["nmat"], case["dtype"]
        s["A"] = _values((n, K, M) if case["tA"] else (n, M, K), dt, gen)
        s["B"] = _values((n, N, K) if case["tB"] else (n, K, N), dt, gen)
        s["C"] = _values((n, M, N), dt, gen)
    else:
        s["A"] = _stored(M, K, case["tA"], case["pad"], case["dtype"], gen)
        s["B"] = _stored(K, N, case["tB"], case["pad"], case["dtype"], gen, weights=case["tB"] == 1)
        if case["packed"]:
            s["packed"] = torch.empty(B.gemm_packed_b_bytes(K, N) // 2, dtype=torch.bfloat16, device="cuda")
            B.gemm_pack_b_bf16(case["tB"], K, N, s["B"], s["B"].shape[1], s["packed"])
        dt = _out_dtype(case)
        s["C"] = (torch.zeros((M, N), dtype=dt, device="cuda") if dt == torch.int32
                  else torch.randn((M, N), device="cuda", generator=gen).to(dt))
        s["bias"] = torch.randn(N, device="cuda", generator=gen) if case["bias"] else None
        s["ws"] = _workspace(B.DTYPE_F32 if case["dtype"] == "f32" else B.DTYPE_BF16, M, N, K, 1)
    return s


def _workspace(dtype, M, N, K, batch):
    return torch.empty(min(B.gemm_workspace_bytes(dtype, M, N, K, batch), WORKSPACE_CAP), dtype=torch.uint8,
                       device="cuda")


# ------------------------------------------------------------------ one pass

def run(s):
    c, C = s["case"], s["C"]
    M, N, K = c["M"], c["N"], c["K"]
    if c["kind"] == "brgemm":
        B.brgemm_bf16(0, 0, M, N, K, c["batch"], s["pool"], s["A_off"], K, s["pool"], s["B_off"], N, c["beta"],
                      C, N, workspace=s["ws"])
        return C
    A, W = s["A"], s["B"]
    lda, ldb = A.shape[-1], W.shape[-1]
    if c["kind"] == "batched":
        n = c["nmat"]
        if c["dtype"] == "f32":
            B.gemm_f32_batched(c["tA"], c["tB"], M, N, K, n, A, lda, M * K, W, ldb, K * N, c["beta"], C, N, M * N)
        else:
            B.gemm_bf16_batched(c["tA"], c["tB"], M, N, K, n, A, lda, M * K, W, ldb, K * N, c["beta"], C, N, M * N, 0)
        return C
    dt = c["dtype"]
    epilogue = (B.EPI_BIAS if c["bias"] else 0) | (B.EPI_RELU if c["relu"] else 0)
    if c["packed"]:
        B.gemm_bf16_packed(c["tA"], M, N, K, A, lda, s["packed"], c["beta"], C, N, c["c32"], s["bias"], epilogue,
                           workspace=s["ws"])
    elif epilogue:
        B.brgemm_fused(B.DTYPE_BF16, c["tA"], c["tB"], M, N, K, 1, A, None, lda, W, None, ldb, c["beta"], C, N,
                       c["c32"], s["bias"], epilogue, workspace=s["ws"])
    elif dt == "f32":
        B.gemm_f32(c["tA"], c["tB"], M, N, K, A, lda, W, ldb, c["beta"], C, N, workspace=s["ws"])
    elif dt == "s8":
        B.gemm_s8(c["tA"], c["tB"], M, N, K, A, lda, W, ldb, 0, C, N)
    else:
        call = {"bf16": B.gemm_bf16, "f16": B.gemm_f16, "f8": B.gemm_f8, "bf8": B.gemm_bf8}[dt]
        call(c["tA"], c["tB"], M, N, K, A, lda, W, ldb, c["beta"], C, N, c["c32"], workspace=s["ws"])
    return C


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    n = case.get("nmat", 1)
    reduce = case.get("batch", 1)
    if case["kind"] == "brgemm":
        esz, csz = 2, 4
    elif case["kind"] == "batched":
        esz = csz = 4 if case["dtype"] == "f32" else 2
    else:
        esz = {"f32": 4, "bf16": 2, "f16": 2}.get(case["dtype"], 1)
        csz = 4 if case["c32"] else 2
    c_passes = 2 if case.get("beta", 0.0) != 0.0 else 1
    moved = n * (reduce * (M * K + K * N) * esz + M * N * csz * c_passes) + (4 * N if case.get("bias") else 0)
    return {"bytes": float(moved), "flops": 2.0 * n * reduce * M * N * K}


def tolerance(case):
    """Largest relative error (2-norm) of another correct implementation.  A 16-bit result carries
    one rounding (bf16 1.7e-3, binary16 2.1e-4 against 64 bits); an fp32 result only the order of
    its fp32 sums (up to 9e-7 at these sizes), and for one-byte floats the matrix instruction's alignment of a group's products
    (1.3e-5).  Integers are exact."""
    dt = case.get("dtype", "bf16")
    if dt == "s8":
        return "exact"
    c32 = case["kind"] == "brgemm" or dt == "f32" or case.get("c32", False)
    if c32:
        return {"rel": 6e-5} if dt in ("f8", "bf8") else {"rel": 4e-6}
    return {"rel": 1e-3} if dt == "f16" else {"rel": 7e-3}


def exact(case, seed):
    s = prepare(case, seed)
    M, N, K, beta = case["M"], case["N"], case["K"], case["beta"]

    def wide(t):
        return t.float().double() if t.dtype.itemsize == 1 and t.dtype.is_floating_point else t.double()

    C0 = wide(s["C"])
    if case["kind"] == "brgemm":
        out = beta * C0 if beta else torch.zeros_like(C0)
        for a, b in zip(s["A_off"].tolist(), s["B_off"].tolist()):
            out += wide(s["pool"][a:a + M * K].reshape(M, K)) @ wide(s["pool"][b:b + K * N].reshape(K, N))
        return out

    def product(a, b):
        a, b = (a[:, :M].t() if case["tA"] else a[:, :K]), (b[:, :K].t() if case["tB"] else b[:, :N])
        return wide(a).contiguous() @ wide(b).contiguous()

    if case["kind"] == "batched":
        out = torch.stack([product(s["A"][z], s["B"][z]) for z in range(case["nmat"])])
    else:
        out = product(s["A"], s["B"])
    if beta:
        out += beta * C0
    if case.get("bias"):
        out += s["bias"].double()
    if case.get("relu"):
        out = out.clamp_min(0.0)
    return out.round().to(torch.int64) if case.get("dtype") == "s8" else out
