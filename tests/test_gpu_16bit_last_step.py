"""The last K-step of 16-bit operands that nothing aligns: chunks over the end of a row are read from further back and moved to
the front.  Every remainder of K and of the rows modulo a chunk, extents of seven to nine elements (on both sides of the
least that can be read back), K within one step, partitions of K, with NaN behind every row, against the oracle."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu

# 64 x 16 tiles of K-step 128 (with K partitions: 38), 64 x 64 of K-steps 64 and 128, 128 x 128, 256 x 256
MEMBERS = (13, 38, 8, 27, 47, 45)


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype,nan", [("bf16", 0x7FC0), ("f16", 0x7E00)])
def test_every_remainder(gpu, dtype, nan, layout):
    sizes = [(7, 8, 9), (8, 7, 8), (9, 9, 7), (8, 8, 8)]
    sizes += [(64 + r, 137 - r, k + r) for k in (8, 120, 256) for r in range(1, 9)] + [(66, 23, 1541), (23, 66, 1027)]
    for s, (M, N, K) in enumerate(sizes):
        p = wl.make_problem(dtype, *layout, M, N, K, alpha=1.5, beta=-0.5, seed=97, key=s, dist="normal",
                            pad=(1 + s % 3, 1 + (s + 1) % 3, s % 3))
        ref, tol = gpu.oracle_full(p), tolerance(p)
        for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
            buf.reshape(-1, ld)[:, cols:] = nan
        dp = gpu.DeviceProblem(p)
        for kid in MEMBERS:
            err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
            assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_whole_chunks_in_unaligned_rows(gpu, layout):
    """Sizes that are multiples of a chunk, one of them not, and all but one: both forms of the step on either side of the rule."""
    for s, (M, N, K) in enumerate([(8, 8, 8), (72, 136, 264), (136, 72, 1032), (72, 136, 265), (71, 136, 264), (72, 135, 264),
                                   (264, 520, 200)]):
        p = wl.make_problem("bf16", *layout, M, N, K, alpha=1.5, beta=-0.5, seed=96, key=s, dist="normal", pad=(3, 1, 2))
        ref, tol = gpu.oracle_full(p), tolerance(p)
        for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
            buf.reshape(-1, ld)[:, cols:] = 0x7FC0
        dp = gpu.DeviceProblem(p)
        for kid in MEMBERS:
            err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
            assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
