"""A selecting call gives the bits of the same call with the member that ks_select names, at sizes where the
count of tiles per compute unit corrects the tree (and beside them): with and without scratch, on aligned rows
and on rows that nothing aligns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {
    "f32": [(0, 0, 6272, 704, 576), (0, 1, 3312, 888, 320), (0, 0, 17956, 1067, 15), (0, 0, 25088, 288, 1152),
            (0, 0, 12544, 576, 1152)],
    "bf16": [(0, 1, 2048, 2048, 2048), (1, 0, 1024, 4096, 4096), (0, 1, 2560, 1280, 1728), (1, 0, 1024, 3712, 5056),
             (0, 1, 2048, 2048, 1920)],
}
SIZES["f16"] = SIZES["bf16"][:3]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_selected_call_has_the_bits_of_the_named_member(dtype):
    import torch
    import gpu_util
    import paper_2003_06795_amd.binding as ks
    kind = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    call = {"f32": ks.gemm_f32, "bf16": ks.gemm_bf16, "f16": ks.gemm_f16}[dtype]
    named = {"f32": ks.gemm_f32_with_kernel, "bf16": ks.gemm_bf16_with_kernel, "f16": ks.gemm_f16_with_kernel}[dtype]
    g = torch.Generator(device="cuda").manual_seed(5)
    try:
        for tA, tB, M, N, K in SIZES[dtype]:
            kid = ks.select(gpu_util.DT[dtype], M, N, K, 1, tA, tB)
            for pad in (0, 3):
                A = (torch.randn((K if tA else M), (M if tA else K) + pad, generator=g, device="cuda") * K ** -0.5).to(kind)
                B = (torch.randn((N if tB else K), (K if tB else N) + pad, generator=g, device="cuda") * K ** -0.5).to(kind)
                for scratch in (None, torch.empty(256 << 20, dtype=torch.uint8, device="cuda")):
                    ks.set_workspace(scratch)
                    C, D = (torch.full((M, N), float("nan"), device="cuda") for _ in range(2))
                    call(tA, tB, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, C, N)
                    named(kid, tA, tB, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, D, N)
                    torch.cuda.synchronize()
                    assert torch.equal(C.view(torch.int32), D.view(torch.int32)), (tA, tB, M, N, K, pad, scratch is None)
                    assert not torch.isnan(C).any()
    finally:
        ks.set_workspace(None)
        gpu_util.ensure_workspace.__defaults__[0].clear()
