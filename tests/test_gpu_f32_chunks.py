"""LDS tiles of K-contiguous fp32 operands ([row][k], four k to a chunk): K at and beside whole chunks, groups of chunks and
K-steps, rows beside the tile, in every load form (multiples of four, of nothing, short and long), against the oracle."""
import numpy as np
import pytest

import workloads as wl
from helpers import tolerance

pytestmark = pytest.mark.gpu

# 16-wide fragments on K-steps of 16, 32 and 64 with one and two K groups, sixteen waves; 32-wide on 16 and 32; balanced
MEMBERS = (21, 31, 7, 61, 28, 29, 32, 47)


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 1)])
def test_k_beside_chunks_and_steps(gpu, layout):
    for s, K in enumerate((1, 3, 4, 7, 8, 15, 16, 17, 31, 32, 33, 36, 63, 64, 65, 127, 129, 300, 324, 641, 1030)):
        M, N = ((65, 36), (64, 128), (131, 260))[s % 3]
        p = wl.make_problem("f32", *layout, M, N, K, batch=1 + s % 2, alpha=1.5, beta=-0.5, seed=95, key=s,
                            pad=(s % 4, (s + 1) % 4, s % 3))
        dp, ref, tol = gpu.DeviceProblem(p), gpu.oracle_full(p), tolerance(p)
        for kid in MEMBERS:
            err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
            assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
