"""The members of 16-bit products with a few rows or columns and of ragged sizes: where the rules beside the built-in tree
take over, both sides of their limits, and that everything else is the tree's."""
import numpy as np
import pytest

import paper_2003_06795_amd.binding as ks


# (type, M, N, K, batch, transA, transB, the tree's member, the member): a size of each rule and one beside it
CASES = [
    (ks.F32, 131072, 285, 9, 1, 0, 0, 28, 23),
    (ks.F32, 118336, 79, 36, 1, 0, 0, 28, 28),
    (ks.F32, 138384, 109, 7, 1, 0, 0, 28, 23),
    (ks.F32, 3496, 1888, 16, 1, 0, 1, 28, 28),
    (ks.F32, 63368, 35, 57, 1, 0, 0, 41, 23),
    (ks.F32, 928, 448, 304, 1, 1, 0, 41, 41),
    (ks.F32, 23716, 108, 27, 1, 0, 0, 41, 23),
    (ks.F32, 10816, 89, 72, 1, 0, 0, 41, 41),
    (ks.F32, 784, 1572, 198, 1, 0, 0, 32, 41),
    (ks.F32, 360, 1768, 384, 1, 1, 0, 32, 32),
    (ks.F32, 315, 2963, 249, 1, 0, 0, 32, 41),
    (ks.F32, 3032, 272, 280, 1, 0, 1, 32, 32),
    (ks.F32, 33, 2180, 2769, 1, 1, 1, 30, 41),
    (ks.F32, 274, 1748, 418, 1, 0, 1, 30, 30),
    (ks.F32, 70, 1401, 1860, 1, 1, 1, 30, 41),
    (ks.F32, 477, 591, 648, 1, 0, 0, 30, 30),
    (ks.F32, 36, 29, 48, 265, 0, 1, 15, 41),
    (ks.F32, 28, 50, 36, 678, 1, 0, 15, 15),
    (ks.F32, 32, 30, 17, 364, 1, 0, 15, 41),
    (ks.F32, 34, 48, 10, 302, 0, 1, 15, 15),
    (ks.F32, 44, 60, 64, 300, 1, 1, 38, 41),
    (ks.F32, 60, 48, 64, 206, 0, 1, 38, 38),
    (ks.F32, 20, 36, 44, 765, 0, 1, 38, 41),
    (ks.F32, 16, 36, 55, 575, 0, 0, 38, 38),
    (ks.F32, 44, 64, 64, 2830, 0, 1, 21, 28),
    (ks.F32, 64, 64, 44, 1175, 0, 1, 21, 21),
    (ks.F32, 52, 52, 55, 3274, 1, 1, 21, 28),
    (ks.F32, 61, 40, 61, 1120, 1, 0, 21, 21),
    (ks.BF16, 2319, 4402, 1025, 1, 1, 0, 23, 45),
    (ks.BF16, 3072, 2048, 1664, 1, 0, 0, 23, 23),
    (ks.BF16, 1434, 7807, 1343, 1, 1, 1, 23, 45),
    (ks.BF16, 1856, 2944, 2752, 1, 0, 0, 23, 23),
    (ks.BF16, 5113, 5712, 1304, 1, 0, 1, 7, 45),
    (ks.BF16, 6720, 3712, 1536, 1, 1, 1, 7, 7),
    (ks.BF16, 8135, 3481, 1199, 1, 0, 1, 7, 45),
    (ks.BF16, 6080, 5440, 1024, 1, 1, 0, 7, 7),
    (ks.BF16, 1024, 2368, 2432, 1, 0, 0, 27, 47),
    (ks.BF16, 320, 320, 58112, 1, 1, 0, 27, 27),
    (ks.BF16, 1919, 1530, 2450, 1, 1, 1, 27, 47),
    (ks.BF16, 1088, 1536, 4288, 1, 0, 1, 27, 27),
]


def tree(M, N, K, tA, tB):
    return int(ks.tune_predict(ks.get_selector(ks.BF16), ks.features(M, N, K, 1, tA, tB)[None])[0])


def rule(M, N, K, tA, tB):
    """Restated: 38 and 13 are 64 x 16 tiles with and without a K split, 27 and 39 square ones of 64."""
    was = tree(M, N, K, tA, tB)
    if K < 1024:
        return was
    if M >= 1024 and N <= 32:
        whole_tt = tA and tB and M % 8 == 0 and K % 8 == 0
        if (N <= 16 and was == 27 and not whole_tt) or (N <= 16 and was == 13 and K >= 1792) or \
                (was == 39 and (N <= 16 or not whole_tt)):
            return 38
    elif M <= 32 and N >= 1024 and K >= 2048:
        if (was in (38, 39) and N >= 1536) or (was == 13 and M <= 16 and N < 8192):
            return 27
    return was


@pytest.mark.parametrize("dtype", [ks.BF16, ks.F16])
def test_rule_and_its_limits(dtype):
    r, seen = np.random.default_rng(3), {}
    few = (1, 2, 7, 8, 15, 16, 17, 31, 32, 33)
    wide = (512, 1023, 1024, 1535, 1536, 2048, 4095, 8191, 8192, 16384)
    deep = (512, 1023, 1024, 1791, 1792, 2047, 2048, 4096, 5041, 8192, 16384, 65536)
    for f in few:
        for w in wide:
            for K in deep:
                tA, tB = int(r.integers(0, 2)), int(r.integers(0, 2))
                for M, N in ((w, f), (f, w)):
                    got, want = ks.select(dtype, M, N, K, 1, tA, tB), rule(M, N, K, tA, tB)
                    assert got == want, (M, N, K, tA, tB)
                    seen[(tree(M, N, K, tA, tB), got)] = 1
                    assert ks.select(dtype, M, N, K, 2, tA, tB) == int(ks.tune_predict(
                        ks.get_selector(ks.BF16), ks.features(M, N, K, 2, tA, tB)[None])[0])
    assert {(27, 38), (13, 38), (39, 38), (38, 27), (13, 27)} <= set(seen)


def test_calls_without_scratch_keep_what_gains_unsplit():
    ptr = 1 << 20                                                        # never dereferenced

    def plan(M, N, K):
        return ks.gemm_plan(ks.BF16, -1, 0, 1, M, N, K, 1.0, ptr, K, ptr, K, 0.0, ptr, N)["kernel_id"]
    try:
        for (M, N, K), without in (((6, 6163, 5041), 38), ((12, 3000, 2100), 13), ((5000, 7, 2100), 13), ((8192, 1, 8192), 38)):
            ks.set_workspace(None)
            assert plan(M, N, K) == without, (M, N, K)
            ks.set_workspace(ptr, 256 << 20)
            assert plan(M, N, K) == ks.select(ks.BF16, M, N, K, 1, 0, 1) == (38 if N < M else 27), (M, N, K)
    finally:
        ks.set_workspace(None)


def test_scratch_that_holds_fewer_partitions_is_none():
    """The rules that count on a K split are timed with all the partitions of the estimate; with less scratch the call keeps
    the member it has without any."""
    ptr = 1 << 20                                                        # never dereferenced

    def plan(M, N, K, kid=-1):
        return ks.gemm_plan(ks.BF16, kid, 0, 1, M, N, K, 1.0, ptr, K, ptr, K, 0.0, ptr, N)
    try:
        for M, N, K in ((6, 6163, 5041), (12, 3000, 2100), (5000, 7, 2100), (8192, 1, 8192), (5, 4096, 16384)):
            ks.set_workspace(None)
            without = plan(M, N, K)["kernel_id"]
            ks.set_workspace(ptr, 256 << 20)
            full = plan(M, N, K)
            # partitions of the member: these calls run in the K-slices form, which stands in for it without any
            used = 4 * M * N * plan(M, N, K, full["kernel_id"])["split_k"]
            assert full["kernel_id"] == ks.select(ks.BF16, M, N, K, 1, 0, 1) and used > 4 * M * N
            for size in (4096, 65536, used - 4, used):
                ks.set_workspace(ptr, size)
                assert plan(M, N, K)["kernel_id"] == (full["kernel_id"] if size >= used else without), (M, N, K, size)
    finally:
        ks.set_workspace(None)


def test_tiles_that_sizes_fit():
    for dtype, M, N, K, batch, tA, tB, was, now in CASES:
        got = int(ks.tune_predict(ks.get_selector(dtype), ks.features(M, N, K, batch, tA, tB)[None])[0])
        assert (got, ks.select(dtype, M, N, K, batch, tA, tB)) == (was, now), (dtype, M, N, K, batch, tA, tB)


# (type, M, N, K, batch, transA, transB, the tree's member): sizes that the larger tile pads to much more, and 16-bit
# ones that are whole multiples of eight with an end of K of their own
PADDED = [
    (ks.F32, 24, 24, 256, 12000, 0, 0, 21),
    (ks.F32, 29, 112, 49, 7846, 0, 1, 21),
    (ks.F32, 91, 28, 65, 3761, 1, 0, 21),
    (ks.F32, 71, 135, 51, 1856, 1, 0, 21),
    (ks.F32, 37, 42, 61, 327, 0, 0, 38),
    (ks.F32, 179963, 20, 59, 1, 0, 0, 41),
    (ks.F32, 154274, 31, 59, 1, 0, 1, 41),
    (ks.BF16, 65536, 64, 4096, 1, 0, 0, 23),
    (ks.BF16, 131072, 33, 4096, 1, 0, 0, 23),
    (ks.BF16, 34831, 338, 1069, 1, 0, 0, 23),
    (ks.BF16, 33000, 64, 2048, 1, 0, 0, 27),
    (ks.BF16, 272, 12160, 2376, 1, 1, 1, 27),
    (ks.BF16, 152, 18008, 2640, 1, 0, 1, 27),
    (ks.BF16, 4592, 4248, 1640, 1, 0, 0, 7),
    (ks.BF16, 5720, 3176, 1656, 1, 1, 0, 7),
    (ks.BF16, 7904, 1280, 1032, 1, 1, 1, 23),
]


@pytest.mark.parametrize("case", PADDED)
def test_larger_tiles_only_where_they_fit(case):
    dtype, M, N, K, batch, tA, tB, member = case
    assert int(ks.tune_predict(ks.get_selector(dtype), ks.features(M, N, K, batch, tA, tB)[None])[0]) == member
    assert ks.select(dtype, M, N, K, batch, tA, tB) == member


def test_a_callers_tree_is_followed():
    leaf = np.zeros(1, dtype=ks.TREE_DTYPE)
    leaf[0] = (-1, 0, 0, 27, 0)
    try:
        ks.set_selector(ks.BF16, leaf)
        assert ks.select(ks.BF16, 8192, 1, 8192) == 27
    finally:
        ks.set_selector(ks.BF16, None)
    assert ks.select(ks.BF16, 8192, 1, 8192) == 38
