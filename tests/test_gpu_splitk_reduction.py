"""The pass that adds the K partitions of a split launch: outputs of one column and of every remainder of four, rows that
fill a work-group's block or not, counts of partitions on both sides of what a group of lanes takes at once, C with and
without 16-byte rows, batches, bias and an output kept in bf16, against the oracle."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance
from oracle import gemm as og

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    import paper_2003_06795_amd.binding as ks
    gpu_util.ensure_workspace(64 << 20)
    yield gpu_util
    ks.set_split_partitions(0)


@pytest.mark.parametrize("partitions", [2, 3, 4, 5, 7, 8, 13, 16, 31, 33, 64])
def test_partitions_of_every_count(gpu, partitions):
    import paper_2003_06795_amd.binding as ks
    ks.set_split_partitions(partitions)
    kid = next(i for i in range(64) if ks.kernel_info(ks.F32, i)["split_k"] == 0 and ks.kernel_info(ks.F32, i)["bk"] == 16)
    for s, (M, N, batch) in enumerate([(1, 1, 1), (3, 4, 2), (65, 6, 1), (5, 259, 3), (130, 132, 1), (9, 1028, 1), (520, 512, 1)]):
        p = wl.make_problem("f32", s % 2, 1 - s % 2, M, N, 2 * 32 * partitions + 5, batch=batch, alpha=1.5,
                            beta=(0.0, -0.5)[s % 2], seed=99, key=s, pad=(0, 0, s % 3))
        dp = gpu.DeviceProblem(p)
        err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - gpu.oracle_full(p))))
        assert err <= tolerance(p), (partitions, (M, N, batch), err)


@pytest.mark.parametrize("N", [64, 70])
@pytest.mark.parametrize("out16", [False, True])
def test_bias_and_bf16_output(gpu, N, out16):
    import torch
    import paper_2003_06795_amd.binding as ks
    ks.set_split_partitions(9)
    p = wl.make_problem("bf16", 0, 1, 37, N, 4096, alpha=1.5, beta=-0.5, seed=99, key=N, dist="normal")
    dp = gpu.DeviceProblem(p)
    bias = wl.uniform_pm1(N, 99, 9, 0)
    ref = p.C0.copy()
    C = dp.C0.bfloat16() if out16 else dp.C0.clone()
    if out16:
        ref = C.float().cpu().numpy()
    og.gemm_bias(p.dtype, p.transA, p.transB, p.M, p.N, p.K, p.alpha, p.A, p.lda, p.B, p.ldb, p.beta, ref, p.ldc, bias)
    call = ks.gemm_out_bf16 if out16 else ks.gemm_bias
    call(ks.BF16, 39, p.transA, p.transB, p.M, p.N, p.K, p.alpha, dp.A, p.lda, dp.B, p.ldb, p.beta, C, p.ldc,
         torch.from_numpy(bias).cuda())
    err = np.abs(C.float().cpu().numpy().astype(np.float64) - ref)
    # the bound of the product, one fp32 rounding more, and for bf16 one step (2^-7) of the value
    assert np.all(err <= tolerance(p) + 2.0 ** -20 + (np.abs(ref) * 2.0 ** -7 if out16 else 0)), float(err.max())


def test_bits_do_not_depend_on_where_the_scratch_lies(gpu):
    """The scratch may be aligned to four bytes only: the same partitions, added in the same order."""
    import torch
    import paper_2003_06795_amd.binding as ks
    ks.set_split_partitions(31)
    scratch = torch.empty((8 << 20) + 16, dtype=torch.uint8, device="cuda")
    for dtype, kid in (("f32", next(i for i in range(64) if ks.kernel_info(ks.F32, i)["split_k"] == 0)), ("bf16", 39)):
        p = wl.make_problem(dtype, 0, 1, 130, 132, 8192, alpha=1.5, beta=-0.5, seed=99, key=5)
        dp, got = gpu.DeviceProblem(p), []
        for at in (0, 4, 8):
            C = dp.C0.clone()
            ks.gemm_with_workspace(gpu.DT[dtype], kid, p.transA, p.transB, p.M, p.N, p.K, p.alpha, dp.A, p.lda, dp.B, p.ldb,
                                   p.beta, C, p.ldc, scratch[at:at + (8 << 20)])
            got.append(C.cpu().numpy())
        assert float(np.max(np.abs(got[0].astype(np.float64) - gpu.oracle_full(p)))) <= tolerance(p)
        assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2]), dtype
    ks.set_split_partitions(0)
