"""The K-slices form of the 16-bit products against fp64: every tile of it in every layout, on aligned operands and on others (odd
sizes, padded rows, addresses inside sixteen bytes), edges of tiles in both directions, K-steps that do not deal out evenly over the waves (and fewer of them than waves), old values, bias, a bf16 output, both 16-bit types, infinities, NaN beside the operands and
operands that are loaded past the last-level cache."""
import pytest

pytestmark = pytest.mark.gpu

# M, N, K: small ones, edges of 16 .. 64 in either direction, one to seventeen K-steps of 64 for the waves, wide operands
SIZES = [(128, 128, 1024), (120, 72, 2048), (8, 8, 576), (1, 24, 1088), (200, 1000, 1536), (1000, 200, 1152), (520, 504, 2112),
         (1024, 1000, 1024), (1000, 1016, 2048), (4096, 8, 1024), (16, 4000, 2048), (6000, 32, 1024), (32, 5000, 2048), (3200, 24, 576),
         (12000, 16, 1024), (24, 9000, 2048), (8, 16384, 1024), (40, 2040, 4096), (7000, 40, 2048), (4584, 8, 512), (1880, 8, 576),
         (1248, 8, 512), (9272, 8, 1216), (3144, 8, 512), (3464, 8, 576), (8, 3464, 576), (4936, 72, 1024), (5000, 64, 960), (3536, 72, 704),
         (1896, 144, 768), (3368, 152, 3008), (1144, 456, 1984), (2208, 264, 3840), (3032, 176, 2496)]


# the same for operands that nothing aligns: ends of K in every place of a chunk, a K-step of which one k is left, short edges
ODD_SIZES = [(127, 129, 1025), (121, 71, 2047), (9, 7, 575), (1, 23, 1089), (199, 1001, 1537), (1001, 199, 1151), (521, 503, 2113),
             (1000, 777, 1509), (777, 1000, 509), (4095, 9, 1023), (15, 4001, 2044), (6001, 31, 1022), (31, 5003, 2050), (3201, 23, 257),
             (12001, 15, 1027), (23, 9001, 2041), (7, 16383, 1021), (41, 2041, 4091), (7001, 39, 2042), (1871, 149, 769), (3001, 170, 1301),
             (64, 64, 2052), (250, 250, 300), (65, 33, 8193), (2500, 64, 700), (48, 3000, 500), (1300, 130, 330), (130, 1300, 330),
             (4517, 10, 300), (4111, 12, 317), (8205, 19, 322), (8331, 18, 444), (9, 4147, 307), (13, 4256, 335)]


def operands(torch, g, tA, tB, M, N, K, kind, pad=0, offset=0):
    """rows of a wider buffer, `offset` elements from its beginning, with NaN in front, between and behind"""
    def one(rows, cols, scale):
        flat = torch.full((offset + rows * (cols + pad) + 8,), float("nan"), device="cuda", dtype=kind)
        view = flat[offset:offset + rows * (cols + pad)].view(rows, cols + pad)
        view[:, :cols] = torch.randn((rows, cols), generator=g, device="cuda").mul_(scale)
        return view
    return one(*((K, M) if tA else (M, K)), K ** -0.5), one(*((N, K) if tB else (K, N)), K ** -0.5)


def product(tA, tB, M, N, K, A, B):
    """op(A) op(B) in fp64 and the bound on its fp32 sums: K exact products, at most K + 16 roundings of 2^-24 of the sum of magnitudes"""
    a = (A[:, :M].t() if tA else A[:, :K]).double().contiguous()
    b = (B[:, :K].t() if tB else B[:, :N]).double().contiguous()
    return a @ b, (a.abs() @ b.abs()) * (K + 16) * 2.0 ** -24


@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("aligned", [True, False])
def test_against_fp64(tA, tB, aligned, kind):
    import torch
    import paper_2003_06795_amd as ks
    g = torch.Generator(device="cuda").manual_seed(7 + 2 * tA + tB)
    dtype, element = {"bf16": (ks.BF16, torch.bfloat16), "f16": (ks.F16, torch.float16)}[kind]
    tiles = set()
    for i, (M, N, K) in enumerate(SIZES if aligned else ODD_SIZES):
        if aligned and ((tA and M % 8) or (not tB and N % 8)):
            continue
        A, B = operands(torch, g, tA, tB, M, N, K, element, *((64 * (i % 5 == 2), 0) if aligned else (i % 4, i % 3)))
        ldc = N + (0, 1, 4)[i % 3]
        # every tile meets each of them: its sizes lie at other places of the list
        epilogue = i + 2 * tA + tB
        out16, beta, with_bias = epilogue % 2 == 1, (0.0, 0.5)[epilogue // 2 % 2], epilogue // 4 % 2 == 1
        C0 = torch.rand((M, ldc), generator=g, device="cuda").mul_(2).sub_(1)
        C = C0.bfloat16() if out16 else C0.clone()
        old = C.double()
        if beta == 0:
            C[:, :N] = float("nan")                       # not read
        bias = torch.rand(N, generator=g, device="cuda")
        args = (tA, tB, M, N, K, 1.5, A, A.shape[1], B, B.shape[1], beta, C, ldc)
        plan = ks.binding.gemm_plan(dtype, -1, *args)
        if plan["path"] < 16:
            continue
        tiles.add(plan["path"] - 16)
        if out16:
            ks.gemm_out_bf16(dtype, -1, *args, bias if with_bias else None)
        elif with_bias:
            ks.gemm_bias(dtype, -1, *args, bias)
        else:
            (ks.gemm_bf16 if dtype == ks.BF16 else ks.gemm_f16)(*args)
        torch.cuda.synchronize()
        want, bound = product(tA, tB, M, N, K, A, B)
        want = 1.5 * want + beta * old[:, :N] + (bias.double() if with_bias else 0)
        bound = 1.5 * bound + 3 * 2.0 ** -24 * (want.abs() + 2) + 1e-12                  # and three roundings of the epilogue
        if out16:
            bound = bound + 2.0 ** -8 * (want.abs() + bound)
        assert bool(((C[:, :N].double() - want).abs() <= bound).all()), (M, N, K, plan["path"])
        assert torch.equal(C[:, N:].double(), old[:, N:])
    assert tiles == (set(range(10)) if aligned else set(range(10, 19))), tiles


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(520, 504, 2112), (503, 521, 2113), (9, 4147, 307), (4111, 12, 317)])
def test_infinities_and_nan_stay_in_their_rows_and_columns(tA, tB, M, N, K):
    """at the last k, in the last row and the last column, which clamped reads repeat, and at the first"""
    import torch
    import paper_2003_06795_amd as ks
    g = torch.Generator(device="cuda").manual_seed(11)
    A, B = operands(torch, g, tA, tB, M, N, K, torch.bfloat16, 0 if K % 64 == 0 else 1)
    at = lambda t, outer, k: (k, outer) if t else (outer, k)
    A[at(tA, M - 1, K - 1)] = float("inf")
    A[at(tA, 3, 0)] = float("nan")
    B[at(not tB, N - 1, K - 1)] = float("-inf")
    B[at(not tB, 2, K // 2)] = float("inf")
    C = torch.empty((M, N), device="cuda")
    args = (tA, tB, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, C, N)
    assert ks.binding.gemm_plan(ks.BF16, -1, *args)["path"] >= 16
    ks.gemm_bf16(*args)
    want, bound = product(tA, tB, M, N, K, A, B)
    got, finite = C.double(), torch.isfinite(want)
    assert int((~finite).sum()) == 2 * N + 2 * M - 4
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
    assert bool(((got - want).abs() <= bound + 1e-12)[finite].all())


def test_operand_past_the_last_level_cache():
    import torch
    import paper_2003_06795_amd as ks
    g = torch.Generator(device="cuda").manual_seed(3)
    for tA, tB, M, N, K in ((0, 0, 8192, 16, 6720), (0, 1, 8, 8000, 6912)):
        A, B = operands(torch, g, tA, tB, M, N, K, torch.bfloat16)
        C = torch.full((M, N), float("nan"), device="cuda")
        args = (tA, tB, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, C, N)
        assert ks.binding.gemm_plan(ks.BF16, -1, *args)["path"] >= 16 and max(M, N) * K * 2 >= 104 << 20
        ks.gemm_bf16(*args)
        want, bound = product(tA, tB, M, N, K, A, B)
        assert bool(((C.double() - want).abs() <= bound + 1e-12).all()), (M, N, K)
