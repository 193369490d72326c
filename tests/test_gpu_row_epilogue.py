"""The epilogue of the two-group 16-bit members on 16x16x32 fragments (ids 44 .. 47), which stores four entries of a row at a time:
edges in the middle of a fragment and of a group of four, outputs that no access of eight or sixteen bytes is aligned to, old
values, bias and a bf16 output, bit for bit against the register-staged path of the same members (one entry per store, the same sums)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kid", [44, 45, 46, 47])
@pytest.mark.parametrize("beta,with_bias,out16", [(0.0, False, False), (0.5, False, False), (-1.25, True, False), (0.0, True, True),
                                                  (0.75, False, True)])
def test_against_the_staged_path(kid, beta, with_bias, out16):
    import torch
    import paper_2003_06795_amd as ks
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * kid + int(8 * beta) + 2 * with_bias + out16)
    for M, N, extra, offset in ((256, 256, 0, 0), (129, 131, 1, 1), (257, 300, 3, 3), (15, 17, 2, 2), (1, 5, 0, 1), (130, 2, 5, 0)):
        K, ldc = 256, N + extra
        A = torch.randn(M, K, generator=g, device="cuda").mul_(K ** -0.5).bfloat16()
        B = torch.randn(N, K, generator=g, device="cuda").mul_(K ** -0.5).bfloat16()
        bias = torch.rand(N + 1, generator=g, device="cuda")[1:] if with_bias else None
        C0 = torch.rand(offset + M * ldc + 64, generator=g, device="cuda").to(torch.bfloat16 if out16 else torch.float32)
        got = []
        for fast in (True, False):
            C = C0.clone()
            args = (ks.BF16, kid, 0, 1, M, N, K, 1.5, A, K, B, K, beta, C[offset:], ldc, bias)
            ks.set_fast_path(fast)
            try:
                (ks.gemm_out_bf16 if out16 else ks.gemm_bias)(*args)
                torch.cuda.synchronize()
            finally:
                ks.set_fast_path(True)
            got.append(C)
        assert torch.equal(got[0], got[1]), (kid, M, N, extra, offset)
        inside = torch.zeros(C0.numel(), dtype=torch.bool, device="cuda")
        inside[offset:offset + M * ldc].view(M, ldc)[:, :N] = True
        assert torch.equal(got[0][~inside], C0[~inside]), (kid, M, N, "wrote beside the matrix")
