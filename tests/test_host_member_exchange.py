"""The members that the count of tiles per compute unit decides between (selector.cpp): every selecting entry
point runs what ks_select names, whatever the operands' alignment and the scratch; where the exchange is made and
where its edges lie; that a caller's own tree, batches and named members are left alone; and that no exchanged
row of the timing tables is slower with the member taken."""
import csv
import glob
import os

import numpy as np
import pytest

import paper_2003_06795_amd as ks

PTR = 1 << 20
DATA = os.path.join(os.path.dirname(ks.binding.__file__), "tune", "data")


def plan(dtype, M, N, K, layout=(0, 1), kid=-1, batch=1, a=PTR, pad=0):
    lda, ldb = (M if layout[0] else K) + pad, (K if layout[1] else N) + pad
    strides = (M * K, K * N, M * N) if batch > 1 else (0, 0, 0)
    return ks.gemm_plan(dtype, kid, *layout, M, N, K, 1.0, a, lda, PTR, ldb, 0.0, PTR, N, batch, *strides)["kernel_id"]


def tree(dtype, M, N, K, batch=1, layout=(0, 1)):
    """What the built-in tree alone says (binary16 runs the 16-bit family with its tree)."""
    dtype = ks.BF16 if dtype == ks.F16 else dtype
    return int(ks.tune_predict(ks.get_selector(dtype), ks.features(M, N, K, batch, *layout)[None])[0])


@pytest.fixture(autouse=True)
def workspace():
    ks.set_workspace(None)
    ks.set_fast_path(True)
    yield
    ks.set_workspace(None)
    ks.set_fast_path(True)
    ks.set_balanced_groups(0)


def test_every_selecting_call_runs_the_member_that_select_names():
    r = np.random.default_rng(7)
    seen = 0
    for n in range(6000):
        dtype = (ks.F32, ks.BF16, ks.F16)[n % 3]
        M, N, K = (int(np.exp(r.uniform(np.log(256), np.log(16384)))) for _ in range(3))
        if n % 2:
            M, N, K = (max(64, v // 64 * 64) for v in (M, N, K))
        layout = (int(r.integers(0, 2)), int(r.integers(0, 2)))
        named = ks.select(dtype, M, N, K, 1, *layout)
        seen += named != tree(dtype, M, N, K, 1, layout)
        if ks.kernel_info(dtype, named)["split_k"] > 1:                     # has a twin for want of scratch
            continue
        for scratch in (0, 1 << 20, 256 << 20):
            ks.set_workspace(PTR, scratch) if scratch else ks.set_workspace(None)
            for a, pad in ((PTR, 0), (PTR + 4, 0), (PTR, 3)):
                assert plan(dtype, M, N, K, layout, a=a, pad=pad) == named, (dtype, M, N, K, layout, scratch, a, pad)
        ks.set_fast_path(bool(n % 4))
        ks.set_balanced_groups(n % 3)
        assert plan(dtype, M, N, K, layout) == named
        ks.set_fast_path(True)
        ks.set_balanced_groups(0)
    assert seen >= 50


def test_one_round_of_two_group_tiles():
    for dtype in (ks.BF16, ks.F16):
        assert tree(ks.BF16, 2048, 2048, 2048) == 23
        assert plan(dtype, 2048, 2048, 2048) == 47
        assert plan(dtype, 2048, 2048, 2048, kid=23) == 23                      # a named member stays
        assert plan(dtype, 2048, 2048, 2048 + 64) != 47                         # half a K-step at the end
        for M, N, K in ((2048, 2048, 1920), (2048 + 128, 2048, 2048), (1024, 2048, 2048)):
            assert plan(dtype, M, N, K) == tree(dtype, M, N, K)


def test_half_k_step_goes_to_the_single_group_member():
    M, N, K = 2560, 1280, 1728
    assert tree(ks.BF16, M, N, K) == 47
    assert plan(ks.BF16, M, N, K) == 9
    assert tree(ks.BF16, 1600, 1216, 5824) == 47                                # both K-contiguous, long K
    assert plan(ks.BF16, 1600, 1216, 5824) == 47


def test_fp32_tiles_that_pad_or_step_badly():
    NN = (0, 0)
    # fewer quarter tiles on the fullest unit, a ragged last column with a short K, padding with a long K
    for M, N, K in ((6272, 704, 576), (17956, 1067, 15), (100352, 32, 1152)):
        assert tree(ks.F32, M, N, K, 1, NN) == 47
        assert plan(ks.F32, M, N, K, NN) == 28
    # as many rounds of either tile; whole columns; no padding
    for M, N, K in ((6272, 512, 576), (12544, 512, 27), (4096, 4096, 4096), (17424, 253, 1926)):
        assert tree(ks.F32, M, N, K, 1, NN) == 47
        assert plan(ks.F32, M, N, K, NN) == 47
    assert plan(ks.F32, 6272, 704, 576, NN, batch=2) == tree(ks.F32, 6272, 704, 576, 2, NN)


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
        was, now = tree(dtype, M, N, K, 1, (tA, tB)), plan(dtype, M, N, K, (tA, tB))
        if was != now and was in t and now in t:
            checked += 1
            assert t[now] <= 1.03 * t[was], (dtype, M, N, K, tA, tB, was, t[was], now, t[now])
    assert checked >= 5
