"""GEMM calls that stand for what programs ask of this library, over the sizes they ask it at.

Sizes come from the repository's workloads: the 128-cube, the fp32 tuning sweep (each dimension
16 .. 4096), im2col convolutions, batched small products and the large / skinny bf16 set.  Where the
tuned sets hold only multiples of 8, odd and unaligned sizes and padded rows are added.

A case is one call of a public entry point:
  entry    gemm (ks.gemm_f32 / gemm_bf16 / gemm_f16), bias (ks.gemm_bias), out16 (ks.gemm_out_bf16, with
           a bias) or own (ks.gemm_with_workspace)
  scratch  whether the program has registered a workspace (256 MiB, as bench.py does); the `own` entry
           passes the same buffer per call instead
  pad      extra elements in every row of A, B and C (operands that are views of wider buffers)
"""
import math

import torch

import paper_2003_06795_amd as ks

WORKSPACE_BYTES = 256 << 20
DTYPES = {"f32": (ks.F32, torch.float32), "bf16": (ks.BF16, torch.bfloat16), "f16": (ks.F16, torch.float16)}
CALLS = {"f32": ks.gemm_f32, "bf16": ks.gemm_bf16, "f16": ks.gemm_f16}
_scratch = []


def _case(dtype, layout, M, N, K, batch=1, alpha=1.0, beta=0.0, entry="gemm", scratch=True, pad=0, name=None):
    case = dict(dtype=dtype, layout=layout, M=M, N=N, K=K, batch=batch, alpha=alpha, beta=beta, entry=entry,
                scratch=scratch, pad=pad)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a single small product, called as in the README: no workspace, latency is all there is
        _case("f32", "NN", 128, 128, 128, scratch=False, name="f32 128 cube"),
        # a small classifier head at a ragged batch: nothing is a multiple of anything
        _case("f32", "NT", 37, 1001, 515, entry="bias", name="f32 ragged head"),
        # a middling layer of the tuning sweep, too few tiles to fill the device without splitting K
        _case("f32", "TN", 480, 1184, 2592, name="f32 split layer"),
        # a 3x3 convolution as im2col: 32 images of 28 x 28, 128 channels in, 256 out
        _case("f32", "NN", 25088, 256, 1152, name="f32 convolution"),
        # the largest fp32 product of the sweep's range, off the tile grid
        _case("f32", "NT", 4095, 3000, 4089, name="f32 large ragged"),
        # batched small products, accumulated at half weight
        _case("f32", "NN", 32, 64, 16, batch=1024, beta=0.5, name="f32 batched"),
        # one decoding step: a weight matrix against sixteen columns
        _case("bf16", "NN", 8192, 16, 8192, name="bf16 skinny"),
        # forward pass of a layer, output kept in bf16, bias fused
        _case("bf16", "NT", 2048, 2048, 2048, entry="out16", name="bf16 layer forward"),
        # weight gradient of the same kind of layer, accumulated over micro-batches
        _case("bf16", "TN", 1024, 4096, 4096, beta=1.0, entry="own", name="bf16 weight gradient"),
        # tall-K reduction into a small matrix
        _case("bf16", "NN", 256, 256, 65536, name="bf16 tall K"),
        # compute-bound square product, prefill of the largest size
        _case("bf16", "NT", 8192, 8192, 8192, name="bf16 large square"),
        # fp16 operands whose rows are not 16-byte aligned
        _case("f16", "NN", 1000, 777, 1509, name="f16 unaligned"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sizes(rng, ranges, cap, step):
    """One size from each range, spread over the logarithm; their product at most `cap`; two thirds of
    the draws on a grid of `step`, as layer widths mostly are."""
    grid = step if rng.random() < 2 / 3 else 1
    while True:
        got = [max(lo, _log_int(rng, lo, hi) // grid * grid) for lo, hi in ranges]
        if math.prod(got) <= cap:
            return got


def draw(rng):
    layout = rng.choice(["NN", "NT", "TN", "TT"])
    pad = rng.choice([0, 0, 0, 8, 3])
    kind = rng.choice(["f32 sweep", "f32 sweep", "f32 convolution", "f32 batched", "16 large", "16 large", "16 skinny",
                       "16 tall", "16 sweep"])
    half = rng.choice(["bf16", "bf16", "f16"])
    entry = rng.choice(["gemm", "gemm", "bias", "out16", "own"])
    if kind == "f32 sweep":
        M, N, K = _sizes(rng, [(16, 4096)] * 3, 2 ** 36, 8)
        return _case("f32", layout, M, N, K, entry=rng.choice(["gemm", "gemm", "bias", "own"]),
                     scratch=rng.random() < 0.8, pad=pad)
    if kind == "f32 convolution":
        images, edge = rng.choice([1, 2, 4, 8, 16, 32]), rng.randint(7, 112)
        N, cin, taps = _log_int(rng, 32, 2048), _log_int(rng, 3, 512), rng.choice([1, 9])
        M, K = images * edge * edge, taps * cin
        while M * N * K > 2 ** 36:
            M //= 2
        return _case("f32", "NN", M, N, K)
    if kind == "f32 batched":
        M, N, K = (rng.randint(1, 16) * 4 if rng.random() < 2 / 3 else rng.randint(4, 64) for _ in range(3))
        return _case("f32", layout, M, N, K, batch=_log_int(rng, 128, 4096), beta=rng.choice([0.0, 0.5]))
    if kind == "16 large":
        M, N, K = _sizes(rng, [(1024, 8192)] * 3, 2 ** 38, 64)
        return _case(half, layout, M, N, K, beta=rng.choice([0.0, 0.0, 1.0]), entry=entry, pad=pad)
    if kind == "16 skinny":
        wide, K = _sizes(rng, [(1024, 16384), (1024, 16384)], 2 ** 27, 128)
        few = _log_int(rng, 1, 256)
        M, N = rng.choice([(wide, few), (few, wide)])
        return _case(half, layout, M, N, K, entry=entry)
    if kind == "16 tall":
        M, N, K = _sizes(rng, [(64, 512), (64, 512), (8192, 65536)], 2 ** 34, 64)
        return _case(half, layout, M, N, K, entry=rng.choice(["gemm", "own"]))
    M, N, K = _sizes(rng, [(64, 4096)] * 3, 2 ** 36, 64)
    return _case(half, layout, M, N, K, entry=entry, scratch=rng.random() < 0.8, pad=pad)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    tA, tB = (int(c == "T") for c in case["layout"])
    M, N, K, batch = case["M"], case["N"], case["K"], case["batch"]
    code, dtype = DTYPES[case["dtype"]]

    def values(rows, cols, kind=dtype):
        """U[-1, 1) for fp32 operands and every output, N(0, 1) / sqrt(K) for 16-bit operands."""
        shape = (batch, rows, cols + case["pad"])
        if kind == torch.float32:
            return torch.rand(shape, generator=g, device="cuda").mul_(2).sub_(1)
        return torch.randn(shape, generator=g, device="cuda").mul_(K ** -0.5).to(kind)

    A = values(K, M) if tA else values(M, K)
    B = values(N, K) if tB else values(K, N)
    C = values(M, N, torch.float32)
    if case["entry"] == "out16":
        C = C.bfloat16()
    bias = values(1, N, torch.float32).reshape(-1)[:N].contiguous() if case["entry"] in ("bias", "out16") else None
    if not _scratch and (case["scratch"] or case["entry"] == "own"):
        _scratch.append(torch.empty(WORKSPACE_BYTES, dtype=torch.uint8, device="cuda"))
    ks.set_workspace(_scratch[0] if case["scratch"] and case["entry"] != "own" else None)
    strides = (A[0].numel(), B[0].numel(), C[0].numel()) if batch > 1 else (0, 0, 0)
    return dict(entry=case["entry"], call=CALLS[case["dtype"]], code=code, C=C, bias=bias, strides=strides, batch=batch,
                head=(tA, tB, M, N, K, case["alpha"], A, A.shape[2], B, B.shape[2], case["beta"], C, C.shape[2]))


def run(state):
    head, batch, strides = state["head"], state["batch"], state["strides"]
    if state["entry"] == "gemm":
        state["call"](*head, batch, *strides)
    elif state["entry"] == "bias":
        ks.gemm_bias(state["code"], -1, *head, state["bias"], batch, *strides)
    elif state["entry"] == "out16":
        ks.gemm_out_bf16(state["code"], -1, *head, state["bias"], batch, *strides)
    else:
        ks.gemm_with_workspace(state["code"], -1, *head, _scratch[0], batch, *strides)
    return state["C"]


def work(case):
    M, N, K, batch = case["M"], case["N"], case["K"], case["batch"]
    operand = 4 if case["dtype"] == "f32" else 2
    out = 2 if case["entry"] == "out16" else 4
    per = (M * K + K * N) * operand + M * N * out * (2 if case["beta"] else 1)
    return {"bytes": batch * per + (4 * N if case["entry"] in ("bias", "out16") else 0), "flops": 2.0 * M * N * K * batch}


def tolerance(case):
    """fp32 sums differ with their order: against an fp64 product of the same operands the relative error
    measured up to 1.1e-6 (K = 4089), single entries up to 9.3e-6.  An output kept in bf16 may land on
    the other side of a rounding boundary: one step of at most 2^-7, 4e-6 of the whole as measured at
    K = 2048 and more of them with a longer K."""
    if case["entry"] == "out16":
        return {"rel": 5e-5, "max": 8e-3}
    return {"rel": 5e-6, "max": 5e-5}
