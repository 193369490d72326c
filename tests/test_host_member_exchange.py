"""The members a launch count decides between (dispatch.hip): where the exchange is made, that its edges lie
where the rule says, and that it leaves alone a caller's own tree, batches, operands off the fast path and the
entry points that name a member."""
import numpy as np
import pytest

import paper_2003_06795_amd as ks

PTR = 1 << 20


def plan(dtype, M, N, K, layout=(0, 1), kid=-1, batch=1, a=PTR):
    lda, ldb = (M if layout[0] else K), (K if layout[1] else N)
    strides = (M * K, K * N, M * N) if batch > 1 else (0, 0, 0)
    return ks.gemm_plan(dtype, kid, *layout, M, N, K, 1.0, a, lda, PTR, ldb, 0.0, PTR, N, batch, *strides)["kernel_id"]


@pytest.fixture(autouse=True)
def workspace():
    ks.set_workspace(None)
    ks.set_fast_path(True)
    yield
    ks.set_workspace(None)


def test_one_round_of_two_group_tiles():
    for dtype in (ks.BF16, ks.F16):
        assert ks.select(dtype, 2048, 2048, 2048, 1, 0, 1) == 23                # what the tree says
        assert plan(dtype, 2048, 2048, 2048) == 47
        assert plan(dtype, 2048, 2048, 2048, kid=23) == 23                      # a named member stays
        assert plan(dtype, 2048, 2048, 2048, a=PTR + 2) == 23                   # off the fast path
        assert plan(dtype, 2048, 2048, 2048 + 64) != 47                         # half a K-step at the end
        assert plan(dtype, 2048, 2048, 1920) != 47 or ks.select(dtype, 2048, 2048, 1920, 1, 0, 1) == 47
        assert plan(dtype, 2048 + 128, 2048, 2048) == ks.select(dtype, 2048 + 128, 2048, 2048, 1, 0, 1)


def test_half_k_step_goes_to_the_single_group_member():
    M, N, K = 2560, 1280, 1728
    assert ks.select(ks.BF16, M, N, K, 1, 0, 1) == 47
    assert plan(ks.BF16, M, N, K) == 9
    assert plan(ks.BF16, M, N, K, a=PTR + 2) == 47


def test_fp32_tiles_that_pad_or_step_badly():
    assert ks.select(ks.F32, 6272, 704, 576, 1, 0, 0) == 47
    assert plan(ks.F32, 6272, 704, 576, (0, 0)) == 28
    assert plan(ks.F32, 4096, 4096, 4096, (0, 0)) == 47
    assert plan(ks.F32, 6272, 704, 576, (0, 0), batch=2) == ks.select(ks.F32, 6272, 704, 576, 2, 0, 0)


def test_a_callers_tree_is_followed():
    leaf = np.zeros(1, dtype=ks.binding.TREE_DTYPE)
    leaf[0] = (-1, 0, 0, 47, 0)
    try:
        ks.set_selector(ks.F32, leaf)
        assert plan(ks.F32, 6272, 704, 576, (0, 0)) == 47
        leaf[0]["value"] = 23
        ks.set_selector(ks.BF16, leaf)
        assert plan(ks.BF16, 2048, 2048, 2048) == 23
    finally:
        ks.set_selector(ks.F32, None)
        ks.set_selector(ks.BF16, None)
    assert plan(ks.F32, 6272, 704, 576, (0, 0)) == 28
