"""16-bit members of K-step 128 on K = 64 (mod 128): the direct-to-LDS path runs the last K-step half, in one
launch, with the same bits as the general path: one half step alone, behind whole ones for every position in
the ring of LDS stages, in the last of several K partitions, and with K beyond that cut off as a remainder."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu

# two, three and four LDS stages, 16- and 32-wide fragments, two groups of waves, split per call and fixed
MEMBERS = (6, 9, 11, 13, 19, 24, 27, 36, 38, 39, 46, 47)


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_half_steps_match_the_general_path_and_the_oracle(gpu, layout):
    import paper_2003_06795_amd.binding as ks
    for s, (M, N, K) in enumerate([(264, 136, 64), (72, 264, 192), (136, 24, 320), (136, 152, 448), (264, 136, 576),
                                   (40, 72, 4160), (136, 264, 600)]):
        dtype = "f16" if s % 3 == 2 else "bf16"
        p = wl.make_problem(dtype, *layout, M, N, K, batch=1 + s % 2, alpha=1.5, beta=-0.5, seed=93, key=s, dist="normal",
                            pad=(8, 0, 3))
        dp = gpu.DeviceProblem(p)
        ref, tol = gpu.oracle_full(p), tolerance(p)
        for kid in MEMBERS:
            plan = ks.gemm_plan(gpu.DT[dtype], kid, *layout, M, N, K, p.alpha, dp.A, p.lda, dp.B, p.ldb, p.beta, dp.C0, p.ldc,
                                p.batch, p.strideA, p.strideB, p.strideC)
            if K % 64 == 0:
                assert plan["path"] >= 1 and plan["k_remainder"] == 0, (kid, plan)
            fast = dp.run(kid)
            err = float(np.max(np.abs(fast.astype(np.float64) - ref)))
            assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
            if plan["k_remainder"] == 0:
                ks.set_fast_path(False)
                try:
                    slow = dp.run(kid)
                finally:
                    ks.set_fast_path(True)
                assert np.array_equal(fast.view(np.uint32), slow.view(np.uint32)), (kid, (M, N, K))
