"""fp32 members on the bf16 matrix pipe (128 x 128 tiles plain and balanced, 64 x 64 with one and two K groups, with and without
K partitions): sizes around the edges of tiles, K-steps and the lines from which the form runs against an fp64 product, its
error against the fp32 pipe's, and operands that it cannot hold, which come out as from fp32 arithmetic."""
import pytest

pytestmark = pytest.mark.gpu

LARGE, PLAIN, SMALL, GROUPS = 47, 59, 28, 32          # (59: the 128 x 128 x 32 member without a balanced form)
UNSPLIT_GROUPS = 13                                   # two K groups, never K partitions
LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


@pytest.fixture()
def ks():
    import torch
    import paper_2003_06795_amd.binding as ks
    import gpu_util
    scratch = torch.empty(68 << 20, dtype=torch.uint8, device="cuda")
    ks.set_workspace(scratch)
    yield ks
    ks.set_split_partitions(0)
    ks.set_workspace(None)
    gpu_util.ensure_workspace.__defaults__[0].clear()


def run(ks, kid, tA, tB, A, B, beta=0.0, C=None, pad=0):
    """op(A) op(B) with rows `pad` elements apart that hold NaN."""
    import torch

    def stored(X, t):
        X = X.t() if t else X
        buf = torch.full((X.shape[0], X.shape[1] + pad), float("nan"), device="cuda")
        buf[:, :X.shape[1]] = X
        return buf
    (M, K), N = A.shape, B.shape[1]
    a, b = stored(A, tA), stored(B, tB)
    C = torch.full((M, N), float("nan"), device="cuda") if C is None else C.clone()
    ks.gemm_f32_with_kernel(kid, tA, tB, M, N, K, 1.0, a, a.shape[1], b, b.shape[1], beta, C, N)
    torch.cuda.synchronize()
    return C


def assert_parts(ks, kid, tA, tB, M, N, K):
    """That the call runs on the bf16 matrix pipe (whatever the operands' alignment)."""
    import torch
    X = torch.empty(16, device="cuda")
    plan = ks.gemm_plan(ks.F32, kid, tA, tB, M, N, K, 1.0, X, M if tA else K, X, K if tB else N, 0.0, X, N)
    assert plan["path"] == 3, (kid, M, N, K, plan)
    return plan


def bound(A, B, K):
    """An MFMA adds sixteen products, each cut off 24 bits below the largest of them and of the accumulator at worst: 2^-22 of
    the sum of magnitudes so far in nearly all cases, once per sixteen k in the accumulator of the large products and five times
    in the one of the small ones, which are 2^-7 of the whole; then one rounding per K group, K partition (64 at
    most) and epilogue step; the products left out are 2^-24 of the whole."""
    return ((K // 16 + 2) * (1 + 5 / 128) * 2.0 ** -22 + (64 + 4 + 1) * 2.0 ** -24) * (A.double().abs() @ B.double().abs())


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid", [LARGE, PLAIN, SMALL, UNSPLIT_GROUPS, GROUPS])
def test_edges(ks, kid, tA, tB):
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    line, on = (360 if kid in (UNSPLIT_GROUPS, GROUPS) else 49), 0
    for n, (M, N, K) in enumerate([(1, 1, 49), (127, 129, 63), (128, 128, 64), (129, 65, 97), (63, 200, 255), (65, 63, 361), (67, 63, 360),
                                   (192, 131, 1025), (3, 260, 2047), (300, 257, 4001), (129, 127, 48), (70, 66, 359)]):
        if kid == GROUPS:
            ks.set_split_partitions(max(1, min(3, K // 400)))
        X = torch.empty(16, device="cuda")
        plan = ks.gemm_plan(ks.F32, kid, tA, tB, M, N, K, 1.0, X, M if tA else K, X, K if tB else N, 0.0, X, N)
        assert plan["path"] == (3 if -(-K // plan["split_k"]) >= line else 0) and (kid == GROUPS or plan["split_k"] == 1)
        on += plan["path"] == 3
        A = torch.rand(M, K, generator=g, device="cuda") * 2 - 1
        B = torch.rand(K, N, generator=g, device="cuda") * 2 - 1
        C0 = torch.rand(M, N, generator=g, device="cuda") if n % 2 else None
        got = run(ks, kid, tA, tB, A, B, 0.5 if n % 2 else 0.0, C0, pad=(0, 3, 8)[n % 3])
        ref = A.double() @ B.double() + (0.5 * C0.double() if n % 2 else 0.0)
        assert ((got.double() - ref).abs() <= bound(A, B, K) + 2.0 ** -23).all(), (kid, M, N, K)
    assert on == (5 if line == 360 else 11)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
def test_two_groups_whose_last_partition_is_one_slice(ks, tA, tB):
    """23 partitions of 368 k, and the four k that are left over: the second K group of the last one has none."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(12)
    M, N, K = 70, 90, 8100
    ks.set_split_partitions(23)
    plan = assert_parts(ks, GROUPS, tA, tB, M, N, K)
    assert plan["split_k"] == 23
    A = torch.rand(M, K, generator=g, device="cuda") * 2 - 1
    B = torch.rand(K, N, generator=g, device="cuda") * 2 - 1
    for at, value in ((K // 3, 0.25), (K - 1, float("inf")), (K // 3, float("inf"))):
        A[3, at] = value
        got, ref = run(ks, GROUPS, tA, tB, A, B), A.double() @ B.double()
        near = ((got.double() - ref).abs() <= bound(A.nan_to_num(0, 1, 1), B, K)) | (got == ref.float()) | (got.isnan() & ref.isnan())
        assert near.all() and got[torch.arange(M, device="cuda") != 3].isfinite().all(), at
        A[3, at] = 0.25


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid", [LARGE, SMALL, UNSPLIT_GROUPS, GROUPS])
def test_what_three_parts_cannot_hold(ks, kid, tA, tB):
    import torch
    g = torch.Generator(device="cuda").manual_seed(4)
    M, N, K = 300, 260, 1100
    if kid == GROUPS:
        ks.set_split_partitions(2)
    plan = assert_parts(ks, kid, tA, tB, M, N, K)
    assert plan["split_k"] == (2 if kid == GROUPS else 1)
    assert_parts(ks, kid, tA, tB, N, M, K)
    A = torch.rand(M, K, generator=g, device="cuda") * 2 - 1
    B = torch.rand(K, N, generator=g, device="cuda") * 2 - 1
    inf, nan, most = float("inf"), float("nan"), torch.finfo(torch.float32).max
    for row, k, value in ((0, 0, inf), (299, 1099, -inf), (130, 700, nan), (70, 33, most), (200, 555, -most)):
        X = A.clone()
        X[row, k] = value
        for swap in (False, True):                           # in either operand
            P, Q = (B.t().contiguous(), X.t().contiguous()) if swap else (X, B)
            got, ref = run(ks, kid, tA, tB, P, Q), P.double() @ Q.double()
            ref32 = ref.float()
            ok = (ref32.isnan() & got.isnan()) | (ref32.isinf() & (got == ref32)) | \
                 (ref32.isfinite() & ((got.double() - ref).abs() <= bound(P.nan_to_num(0, most, -most), Q.nan_to_num(0, most, -most), K)))
            # a sum beyond the largest float may overflow a step earlier or later in another order
            assert ok[ref.abs().nan_to_num(0, 0) < 0.9 * most].all(), (kid, value, swap)
    # sums and operands on both sides of what is held, and magnitudes that are all held
    for scale, other in ((2.0 ** 40, 2.0 ** 34), (2.0 ** 40, 2.0 ** 44), (2.0 ** 104, 2.0 ** -104), (2.0 ** 106, 2.0 ** -106),
                         (2.0 ** -110, 1.0), (2.0 ** -126, 2.0 ** 100), (2.0 ** -140, 2.0 ** 120)):
        X, Y = A * scale, B * other
        ref = X.double() @ Y.double()
        assert ((run(ks, kid, tA, tB, X, Y).double() - ref).abs() <= bound(X, Y, K)).all(), (kid, scale)
    X = A.clone()
    X[17] *= 2.0 ** -120                                     # one small row among ordinary ones, and zeros
    X[40:90] = 0.0
    ref = X.double() @ B.double()
    assert ((run(ks, kid, tA, tB, X, B).double() - ref).abs() <= bound(X, B, K)).all()


@pytest.mark.parametrize("tA,tB", LAYOUTS)
def test_four_tiles_as_one(ks, tA, tB):
    """The unsplit 64 x 64 member on 2 x 2 tiles per work-group: its bits on whole and ragged edges, where the rule takes it, are
    those of single tiles, which a forced count gives."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    try:
        for M, N, K in ((2816, 2560, 80), (2753, 2497, 129), (57000, 97, 96)):
            A, B = torch.rand(M, K, generator=g, device="cuda") - 0.5, torch.rand(K, N, generator=g, device="cuda") - 0.5
            out = {}
            for forced, per in ((1, 1), (0, 4)):
                ks.set_tiles_per_workgroup(forced)
                plan = ks.gemm_plan(ks.F32, SMALL, tA, tB, M, N, K, 1.0, A, M if tA else K, B, K if tB else N, 0.0, A, N)
                edge = 128 if per == 4 else 64
                assert plan["tiles_per_workgroup"] == per and plan["workgroups"] == -(-M // edge) * -(-N // edge)
                out[per] = run(ks, SMALL, tA, tB, A, B, pad=3)
            assert torch.equal(out[1], out[4]), (M, N, K)
            X = A.clone()
            X[70, 3], X[M - 1, K - 1] = float("inf"), 2.0 ** 110
            for forced in (1, 0):
                ks.set_tiles_per_workgroup(forced)
                out[forced] = run(ks, SMALL, tA, tB, X, B, pad=3)
            assert torch.equal(out[1].nan_to_num(7.0), out[0].nan_to_num(7.0)), (M, N, K)
            assert ((out[4].double() - A.double() @ B.double()).abs() <= bound(A, B, K)).all()
    finally:
        ks.set_tiles_per_workgroup(0)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
def test_forced_counts_of_the_64_x_64_member(ks, tA, tB):
    """Four tiles per work-group are 2 x 2 as one wherever the form runs, any other count single tiles; the bits are the same."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(11)
    try:
        for M, N, K in ((1, 1, 49), (65, 130, 79), (127, 64, 100), (200, 257, 192)):
            A, B = torch.rand(M, K, generator=g, device="cuda") - 0.5, torch.rand(K, N, generator=g, device="cuda") - 0.5
            out = {}
            for forced in (1, 2, 4, 64):
                ks.set_tiles_per_workgroup(forced)
                plan = assert_parts(ks, SMALL, tA, tB, M, N, K)
                edge = 128 if forced == 4 else 64
                assert plan["tiles_per_workgroup"] == (4 if forced == 4 else 1)
                assert plan["workgroups"] == -(-M // edge) * -(-N // edge)
                out[forced] = run(ks, SMALL, tA, tB, A, B, pad=3)
            assert all(torch.equal(out[1], out[n]) for n in (2, 4, 64)), (M, N, K)
    finally:
        ks.set_tiles_per_workgroup(0)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid,K", [(PLAIN, 64), (SMALL, 64), (UNSPLIT_GROUPS, 400)])
def test_small_magnitudes_at_every_place(ks, kid, K, tA, tB):
    """One term to a sum, small or subnormal, in each place of a chunk of four k and of four rows or columns.  2^-22: three bf16
    parts hold the operands exactly, the products left out are 2^-24 of the whole, the last rounding as much, and the small
    products' half a unit of 2^-8 of it; 2^-149: the unit of a subnormal sum."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(6)
    M, N = 130, 131
    assert_parts(ks, kid, tA, tB, M, N, K)
    for value, other in ((1.2345678e-35, 1.0), (1.2345678e-39, 1.0), (3e-45, 2.0 ** 60), (1.2345678e-35, 2.0 ** 100)):
        for place in range(4):
            for k in range(4):
                X = torch.zeros(M, K, device="cuda")
                X[place::4, k] = value
                Y = (torch.rand(K, N, generator=g, device="cuda") + 0.5) * other
                for P, Q, t in ((X, Y, 0), (Y.t().contiguous(), X.t().contiguous(), 1)):
                    if t:
                        assert_parts(ks, kid, tA, tB, N, M, K)
                    got, ref = run(ks, kid, tA, tB, P, Q).double(), P.double() @ Q.double()
                    assert ((got - ref).abs() <= 2.0 ** -22 * ref.abs() + 2.0 ** -149).all(), (value, other, place, k, t)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid,K", [(PLAIN, 256), (SMALL, 256), (UNSPLIT_GROUPS, 400)])
def test_products_around_the_smallest_float(ks, kid, K, tA, tB):
    """Operands of ordinary magnitude whose products, or whose sums, are near 2^-126 and below: no part of a product is lost."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    M, N = 130, 131
    assert_parts(ks, kid, tA, tB, M, N, K)
    A = torch.rand(M, K, generator=g, device="cuda") + 0.5
    B = torch.rand(K, N, generator=g, device="cuda") + 0.5
    for a, b in ((-55, -62), (-64, -64), (-90, -40), (-40, -90), (-75, -74), (-130, 1)):
        X, Y = A * 2.0 ** a, B * 2.0 ** b
        ref = X.double() @ Y.double()
        assert ((run(ks, kid, tA, tB, X, Y).double() - ref).abs() <= bound(X, Y, K) + 2.0 ** -149).all(), (a, b)


# rms error over sum |a b| against that of a member on the fp32 matrix pipe (64 x 64 tiles, one K group), at most: measured 0.28 - 0.45,
# 0.35 - 0.60, 0.69 - 0.90, 1.02 - 1.03 and 1.13 - 1.20 of it.  (All six products in one accumulator give 0.8, 0.8, 1.5 - 1.9, 1.35 and 1.0 - 1.2.)
FP32_PIPE = 60
ERRORS = {"dense": 0.55, "positive, uneven": 0.7, "four terms": 1.0, "one term": 1.1, "nearly one term": 1.3}


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid,K", [(PLAIN, 64), (PLAIN, 2048), (LARGE, 1100), (SMALL, 64), (SMALL, 512), (UNSPLIT_GROUPS, 400),
                                   (UNSPLIT_GROUPS, 2048)])
def test_error_is_the_fp32_pipes(ks, kid, K, tA, tB):
    import torch
    g = torch.Generator(device="cuda").manual_seed(8)
    M = N = 384
    ks.set_workspace(None)                                   # one K range to a tile in either member
    assert_parts(ks, kid, tA, tB, M, N, K)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")
    one = torch.zeros(M, K, device="cuda")
    one[torch.arange(M), torch.arange(M) % K] = 1.0
    few = (torch.rand(M, K, generator=g, device="cuda") < 4.0 / K).float()
    for what, A, B in (("dense", torch.rand(M, K, generator=g, device="cuda") * 2 - 1, torch.rand(K, N, generator=g, device="cuda") * 2 - 1),
                       ("positive, uneven", (2 * normal(M, K)).exp(), (2 * normal(K, N)).exp()),
                       ("four terms", few * normal(M, K), normal(K, N)),
                       ("one term", one * normal(M, 1), normal(K, N)),
                       ("nearly one term", torch.softmax(32 * normal(M, K), 1), normal(K, N))):
        ref, whole = A.double() @ B.double(), A.double().abs() @ B.double().abs()
        rms = {}
        for k in (kid, FP32_PIPE):
            error = (run(ks, k, tA, tB, A, B).double() - ref)[whole > 0] / whole[whole > 0]
            rms[k] = error.square().mean().sqrt().item()
        assert rms[kid] <= ERRORS[what] * rms[FP32_PIPE], (what, rms)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid,K", [(PLAIN, 192), (SMALL, 192), (UNSPLIT_GROUPS, 400)])
def test_every_part_arrives(ks, kid, K, tA, tB):
    """Floats of 24 random bits times one power of two each come out as they are: each entry is one operand's three parts."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(9)
    M, N = 150, 170
    assert_parts(ks, kid, tA, tB, M, N, K)
    A = (torch.rand(M, K, generator=g, device="cuda") + 0.5) * torch.where(torch.rand(M, K, generator=g, device="cuda") < 0.5, -1.0, 1.0)
    B = torch.zeros(K, N, device="cuda")
    at = torch.randint(0, K, (N,), generator=g, device="cuda")
    powers = torch.randint(-20, 20, (N,), generator=g, device="cuda").cpu()
    B[at, torch.arange(N, device="cuda")] = torch.ldexp(torch.ones(N), powers).cuda()
    expected = A[:, at] * B.amax(0)
    assert torch.equal(run(ks, kid, tA, tB, A, B), expected)
    assert_parts(ks, kid, tA, tB, N, M, K)
    assert torch.equal(run(ks, kid, tA, tB, B.t().contiguous(), A.t().contiguous()), expected.t())


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("kid,K", [(LARGE, 1100), (PLAIN, 192), (SMALL, 192), (UNSPLIT_GROUPS, 400)])
def test_other_rows_and_columns_keep_their_bits(ks, kid, K, tA, tB):
    """What an entry's own row and column hold decides how it is computed, not what stands beside them: an infinity, a NaN or a
    float that the parts cannot hold changes the bits of its row or column only, and none of them beyond the matrix changes any."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(10)
    M, N = 300, 270
    assert_parts(ks, kid, tA, tB, M, N, K)
    A = torch.rand(M, K, generator=g, device="cuda") - 0.5
    B = torch.rand(K, N, generator=g, device="cuda") - 0.5
    whole = run(ks, kid, tA, tB, A, B)
    assert torch.equal(run(ks, kid, tA, tB, A, B, pad=3), whole)       # (rows that end in NaN)
    for value in (float("inf"), float("nan"), 2.0 ** 110):
        for row, k in ((0, 0), (77, K - 1), (299, K // 2)):
            X = A.clone()
            X[row, k] = value
            got = run(ks, kid, tA, tB, X, B)
            others = torch.arange(M, device="cuda") != row
            assert torch.equal(got[others], whole[others]), (value, row)
            ref = X.double() @ B.double()
            assert torch.equal(got[row].isnan(), ref[row].float().isnan()) and \
                (not ref[row].isfinite().all() or ((got[row].double() - ref[row]).abs() <= 2.0 ** -18 * (X.double().abs() @ B.double().abs())[row]).all())
        for col, k in ((0, 0), (200, K - 1), (269, K // 2)):
            Y = B.clone()
            Y[k, col] = value
            got = run(ks, kid, tA, tB, A, Y)
            others = torch.arange(N, device="cuda") != col
            assert torch.equal(got[:, others], whole[:, others]), (value, col)
