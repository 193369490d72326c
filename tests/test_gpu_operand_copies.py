"""Aligned copies of 16-bit operands (ks_set_operand_copies): rows and K of every remainder, fewer elements than a chunk,
odd bases and gaps of NaN, one operand or both, against the oracle; the scratch that such a call may and may not use."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu

# 16 columns with a fixed split, 64 x 64 x 128, 128 x 128 and 256 x 256 in two groups of waves; one that never splits
MEMBERS = (26, 27, 47, 45, 13)
SHAPES = [(1, 1, 1), (7, 5, 9), (3, 130, 131), (130, 3, 264), (65, 129, 127), (257, 255, 193), (264, 40, 260), (16, 16, 129),
          (129, 264, 576)]


@pytest.fixture()
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    import paper_2003_06795_amd.binding as ks
    yield gpu_util
    ks.set_operand_copies(-1)
    gpu_util.ensure_workspace.__defaults__[0].clear()
    ks.set_workspace(None)


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_copies_match_the_oracle(gpu, dtype, layout):
    import torch
    import paper_2003_06795_amd.binding as ks
    nan = 0x7FC0 if dtype == "bf16" else 0x7E00
    scratch = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    for s, (M, N, K) in enumerate(SHAPES):
        p = wl.make_problem(dtype, *layout, M, N, K, alpha=1.5, beta=-0.5, seed=97, key=s, dist="normal",
                            pad=(s % 4, (s + 1) % 4, s % 3))
        ref, tol = gpu.oracle_full(p), tolerance(p)
        for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
            buf.reshape(-1, ld)[:, cols:] = nan
        dp = gpu.DeviceProblem(p)
        odd = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:] for t in (dp.A, dp.B)]
        for at, t in zip(odd, (dp.A, dp.B)):
            at.copy_(t)
        for A, B in ((dp.A, dp.B), odd, (dp.A, odd[1])):
            for kid in MEMBERS:
                got = []
                for mode in (0, 1):
                    ks.set_operand_copies(mode)
                    scratch.fill_(0xFF)                                         # NaN wherever it is read unwritten
                    C = dp.C0.clone()
                    ks.gemm_with_workspace(gpu.DT[dtype], kid, p.transA, p.transB, M, N, K, p.alpha, A, p.lda, B, p.ldb,
                                           p.beta, C, p.ldc, scratch[4:])
                    got.append(C.cpu().numpy())
                err = float(np.max(np.abs(got[1].astype(np.float64)[:ref.size] - ref)))
                assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
                assert np.array_equal(got[0], got[1]), (kid, (M, N, K))         # the same sums in the same order


def test_scratch_of_the_copies(gpu):
    import torch
    import paper_2003_06795_amd.binding as ks
    ks.set_operand_copies(1)
    p = wl.make_problem("bf16", 0, 1, 130, 70, 131, alpha=1.0, beta=0.0, seed=98, dist="normal", c_fill="nan")
    dp, ref, tol = gpu.DeviceProblem(p), gpu.oracle_full(p), tolerance(p)
    need = 2 * (130 + 70) * 192 + 16
    args = (p.transA, p.transB, p.M, p.N, p.K, p.alpha, dp.A, p.lda, dp.B, p.ldb, p.beta)
    for kid, own, size, used in ((13, True, need, True), (13, True, need - 1, False), (13, False, need, False),
                                 (45, False, need, True), (45, False, need - 1, False)):
        ws = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        C = dp.C0.clone()
        if own:
            ks.set_workspace(None)
            ks.gemm_with_workspace(ks.BF16, kid, *args, C, p.ldc, ws)
        else:
            ks.set_workspace(ws)
            ks.gemm_bf16_with_kernel(kid, *args, C, p.ldc)
        err = float(np.max(np.abs(C.cpu().numpy().astype(np.float64) - ref)))
        assert err <= tol, (kid, own, size, err)
        assert bool((ws != 0x5A).any()) == used, (kid, own, size)
    for bad in (-2, 2):
        with pytest.raises(ks.KsError):
            ks.set_operand_copies(bad)


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_copies_with_a_hybrid_launch(gpu, layout):
    """272 tiles on 256 units: the copies at the end of the scratch, the partial tiles of the last round at its beginning."""
    import torch
    import paper_2003_06795_amd.binding as ks
    ks.set_operand_copies(1)
    ks.set_tail_split(4)
    try:
        p = wl.make_problem("bf16", *layout, 1085, 1021, 1091, alpha=1.5, beta=-0.5, seed=99, dist="normal", pad=(3, 1, 2))
        dp, ref = gpu.DeviceProblem(p), gpu.oracle_full(p)
        args = (p.transA, p.transB, p.M, p.N, p.K, p.alpha, dp.A, p.lda, dp.B, p.ldb, p.beta)
        copies = 2 * (1088 + 1024) * 1152 + 16
        for size, tail in ((copies + 4 * 16 * 64 * 64 * 4, 4), (copies, 0)):          # with and without room for the partial tiles
            ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
            ks.set_workspace(ws)
            C = dp.C0.clone()
            plan = ks.gemm_plan(ks.BF16, 39, *args, C, p.ldc)
            assert (plan["operand_copies"], plan["tail_split"]) == (3, tail), plan
            ks.gemm_bf16_with_kernel(39, *args, C, p.ldc)
            err = float(np.max(np.abs(C.cpu().numpy()[:ref.size].astype(np.float64) - ref)))
            assert err <= tolerance(p), (size, err)
    finally:
        ks.set_tail_split(-1)
