"""The members a launch count decides between (dispatch.hip): where the exchange is made, that its edges lie
where the rule says, and that it leaves alone a caller's own tree, batches, operands off the fast path and the
entry points that name a member."""
import csv
import glob
import os

import numpy as np
import pytest

import paper_2003_06795_amd as ks

PTR = 1 << 20
DATA = os.path.join(os.path.dirname(ks.binding.__file__), "tune", "data")


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
    NN = (0, 0)
    # fewer quarter tiles on the fullest unit, a ragged last column with a short K, padding with a long K
    for M, N, K in ((6272, 704, 576), (17956, 1067, 15), (100352, 32, 1152)):
        assert ks.select(ks.F32, M, N, K, 1, *NN) == 47
        assert plan(ks.F32, M, N, K, NN) == 28
    # as many rounds of either tile; whole columns; no padding
    for M, N, K in ((6272, 512, 576), (12544, 512, 27), (4096, 4096, 4096), (17424, 253, 1926)):
        assert ks.select(ks.F32, M, N, K, 1, *NN) == 47
        assert plan(ks.F32, M, N, K, NN) == 47
    assert plan(ks.F32, 6272, 704, 576, NN, batch=2) == ks.select(ks.F32, 6272, 704, 576, 2, *NN)


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


def test_no_exchanged_row_of_the_timing_tables_is_slower():
    """3 %: what repeated medians of one cell of the tables differ by.  The 16-bit tables were timed on hot operands
    and hold only whole K-steps for these members."""
    ms = {}
    for path in glob.glob(os.path.join(DATA, "timings_*.csv")):
        dtype = ks.F32 if os.path.basename(path).startswith("timings_f32") else ks.BF16
        for row in csv.DictReader(open(path)):
            if row["median_ms"] and int(row["batch"]) == 1:
                key = (dtype,) + tuple(int(row[c]) for c in ("M", "N", "K", "transA", "transB"))
                ms.setdefault(key, {})[int(row["kernel"])] = float(row["median_ms"])
    checked = 0
    ks.set_workspace(PTR, 1 << 30)
    for (dtype, M, N, K, tA, tB), t in ms.items():
        was, now = ks.select(dtype, M, N, K, 1, tA, tB), plan(dtype, M, N, K, (tA, tB))
        if was != now and was in t and now in t:
            checked += 1
            assert t[now] <= 1.03 * t[was], (dtype, M, N, K, tA, tB, was, t[was], now, t[now])
    assert checked >= 5
