"""The fp32 members read operands that nothing aligns sixteen bytes at a time: every remainder of K
modulo a unit of four, rows of fewer than four elements (where a whole unit would leave the matrix),
extents one off a tile, odd leading dimensions, odd base addresses and rows so long that lane offsets
leave 32 bits, against the oracle.  The gaps between rows hold NaN: what is read there must not reach C."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu

# one member per loader shape and core: FMA, 16x16 fragments with 1 .. 16 waves, K groups, direct, K-sliced,
# multi-tile, split per call, balanced
MEMBERS = (0, 6, 7, 16, 21, 25, 28, 30, 32, 37, 43, 44, 47, 56, 60, 63)
SHAPES = [(1, 1, 1), (7, 5, 9), (2, 130, 131), (130, 3, 131), (65, 129, 34), (257, 255, 193), (127, 40, 260),
          (16, 16, 128), (129, 263, 1030),
          # extents of whole units and a short K: the form with one kind of K-step
          (4, 4, 4), (40, 56, 24), (68, 132, 20), (260, 64, 100)]


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_unaligned_operands_match_the_oracle(gpu, layout):
    import torch
    for s, (M, N, K) in enumerate(SHAPES):
        pad = (s % 4, (s + 1) % 4, s % 3)
        p = wl.make_problem("f32", *layout, M, N, K, batch=1 + s % 2, alpha=1.5, beta=-0.5, seed=92, key=s,
                            dist="uniform", pad=pad)
        ref = gpu.oracle_full(p)
        tol = tolerance(p)
        for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
            buf.reshape(-1, ld)[:, cols:] = np.nan
        dp = gpu.DeviceProblem(p)
        odd = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:] for t in (dp.A, dp.B)]
        for at, t in zip(odd, (dp.A, dp.B)):
            at.copy_(t)
        for A, B in ((dp.A, dp.B), odd):
            dp.A, dp.B = A, B
            for kid in MEMBERS:
                err = np.abs(dp.run(kid).astype(np.float64) - ref)
                assert float(np.max(err)) <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), np.max(err), tol)


def test_rows_longer_than_lane_offsets_reach(gpu):
    import torch
    import paper_2003_06795_amd as ks
    M, N, K, ld = 3, 5, 70, (1 << 22) + 3
    A = torch.empty(M * ld, device="cuda")
    a = torch.rand(M, K, device="cuda") * 2 - 1
    A.view(M, ld)[:, :K] = a
    B = torch.rand(K, N, device="cuda") * 2 - 1
    ref = a.double() @ B.double()
    for kid in MEMBERS:
        C = torch.full((M, N), float("nan"), device="cuda")
        ks.gemm_f32_with_kernel(kid, 0, 0, M, N, K, 1.0, A, ld, B, N, 0.0, C, N)
        assert float((C.double() - ref).abs().max()) <= 1e-5 * K, kid


@pytest.mark.parametrize("few", [1, 2, 3])
def test_rows_shorter_than_a_unit(gpu, few):
    """Row-contiguous operands whose rows of one to three elements lie side by side: a unit of four reaches up to
    three rows ahead, which the last rows do not have."""
    for K in (32, 33, 34, 35, 64, 257, 1030):
        for M, N, layout in ((few, 130, (1, 0)), (few, 130, (1, 1)), (130, few, (0, 0)), (130, few, (1, 0)), (few, few, (1, 0))):
            p = wl.make_problem("f32", *layout, M, N, K, alpha=1.5, beta=-0.5, seed=94, key=K, dist="uniform")
            ref, tol = gpu.oracle_full(p), tolerance(p)
            dp = gpu.DeviceProblem(p)
            for kid in MEMBERS:
                err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
                assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
