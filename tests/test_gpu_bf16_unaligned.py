"""The register-staged path of the 16-bit members reads operands that nothing aligns sixteen bytes at a
time: every remainder of K modulo a chunk of eight, rows of fewer than eight elements (where a whole
chunk would leave the matrix), extents one off a tile, odd leading dimensions and odd base addresses,
against the oracle.  The gaps between rows hold NaN: what is read there must not reach C."""
import numpy as np
import pytest

import workloads as wl
from helpers import operand_matrices, tolerance

pytestmark = pytest.mark.gpu

# one member per loader shape: 16 columns (idle threads), 64 x 64, 128 x 128 with two K-steps in flight, 256 x 256
MEMBERS = (12, 13, 14, 27, 30, 47, 45)
SHAPES = [(1, 1, 1), (7, 5, 9), (3, 130, 131), (130, 3, 131), (65, 129, 127), (257, 255, 193), (127, 40, 260),
          (16, 16, 128), (129, 263, 518)]


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import gpu_util
    gpu_util.ensure_workspace(64 << 20)
    return gpu_util


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_unaligned_operands_match_the_oracle(gpu, dtype, layout):
    import torch
    nan = 0x7FC0 if dtype == "bf16" else 0x7E00
    for s, (M, N, K) in enumerate(SHAPES):
        pad = (s % 4, (s + 1) % 4, s % 3)
        p = wl.make_problem(dtype, *layout, M, N, K, batch=1 + s % 2, alpha=1.5, beta=-0.5, seed=91, key=s,
                            dist="normal", pad=pad)
        ref = gpu.oracle_full(p)
        tol = tolerance(p)
        assert np.all(np.isfinite([m for pair in operand_matrices(p)[:2] for m in map(np.max, pair)]))
        for buf, ld, cols in ((p.A, p.lda, M if p.transA else K), (p.B, p.ldb, K if p.transB else N)):
            buf.reshape(-1, ld)[:, cols:] = nan
        dp = gpu.DeviceProblem(p)
        odd = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:] for t in (dp.A, dp.B)]
        for at, t in zip(odd, (dp.A, dp.B)):
            at.copy_(t)
        for A, B in ((dp.A, dp.B), odd):
            dp.A, dp.B = A, B
            for kid in MEMBERS:
                err = np.abs(dp.run(kid).astype(np.float64) - ref)
                assert float(np.max(err)) <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), np.max(err), tol)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_few_k_steps_of_k_contiguous_operands(gpu, dtype):
    """K a multiple of eight with one to four K-steps of 128, the last one partial: the one-loop form of the members of
    that K-step and, on both sides of its limits, the other one."""
    nan = 0x7FC0 if dtype == "bf16" else 0x7E00
    for s, (M, N, K) in enumerate([(65, 129, 120), (7, 5, 136), (130, 17, 248), (257, 255, 264), (16, 16, 392), (129, 263, 504),
                                   (66, 130, 520)]):
        p = wl.make_problem(dtype, 0, 1, M, N, K, batch=1 + s % 2, alpha=1.5, beta=-0.5, seed=96, key=s, dist="normal",
                            pad=(s % 3, (s + 1) % 4, s % 3))
        ref, tol = gpu.oracle_full(p), tolerance(p)
        for buf, ld in ((p.A, p.lda), (p.B, p.ldb)):
            buf.reshape(-1, ld)[:, K:] = nan
        dp = gpu.DeviceProblem(p)
        for kid in (6, 9, 11, 13, 16, 19, 27, 28, 36, 38, 39, 46, 47):
            err = float(np.max(np.abs(dp.run(kid).astype(np.float64) - ref)))
            assert err <= tol, "kernel %d %s: %.3e > %.3e" % (kid, (M, N, K), err, tol)
