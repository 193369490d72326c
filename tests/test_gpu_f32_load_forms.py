"""The LDS-staged fp32 members fetch a K-step in one of three ways, chosen by the member, the extents and the
number of K-steps: every such member on both sides of each of those limits, with extents that are multiples of
four and with ragged ones, against the oracle.  The gaps between rows hold NaN."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("ragged", [False, True])
def test_every_member_on_both_sides_of_each_limit(gpu, layout, ragged):
    import paper_2003_06795_amd.binding as ks
    members = {}
    for kid in range(ks.num_kernels(ks.F32)):
        ki = ks.kernel_info(ks.F32, kid)
        if ki["core_name"] in ("fma", "mfma16", "mfma32"):
            members.setdefault(ki["bk"] * ki["k_waves"], []).append(kid)
    M, N = (133, 137) if ragged else (136, 132)
    for step, kids in sorted(members.items()):
        for K in (step, step + 4, 2 * step, 2 * step + 4, 8 * step, 8 * step + 4):
            K -= 3 if ragged else 0
            p = wl.make_problem("f32", *layout, M, N, K, alpha=1.5, beta=-0.5, seed=95, key=K, dist="uniform",
                                pad=(1, 2, 3) if ragged else (4, 0, 4))
            ref, tol = gpu.oracle_full(p), tolerance(p)
            for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
                buf.reshape(-1, ld)[:, cols:] = np.nan
            dp = gpu.DeviceProblem(p)
            for kid in kids:
                err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
                assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
