"""The members of 16-bit products with a few rows or columns: where the rule beside the built-in tree takes over, both sides
of each of its limits, and that everything else is the tree's."""
import numpy as np
import pytest

import paper_2003_06795_amd.binding as ks


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
    few = (1, 2, 7, 8, 15, 16, 17, 31, 32, 33, 64)
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


def test_a_callers_tree_is_followed():
    leaf = np.zeros(1, dtype=ks.TREE_DTYPE)
    leaf[0] = (-1, 0, 0, 27, 0)
    try:
        ks.set_selector(ks.BF16, leaf)
        assert ks.select(ks.BF16, 8192, 1, 8192) == 27
    finally:
        ks.set_selector(ks.BF16, None)
    assert ks.select(ks.BF16, 8192, 1, 8192) == 38
