"""Aligned copies of 16-bit operands (ks_set_operand_copies) as the planner decides on them: what the scratch has to hold
beside the copies.  No device: the planner reads sizes, leading dimensions and pointer alignment only."""
import random

import pytest

import paper_2003_06795_amd.binding as ks

PTR = 1 << 20                                   # never dereferenced


@pytest.fixture()
def plan():
    def of(mode, scratch, tA, tB, M, N, K, kid=-1, pad=3, dtype=ks.BF16):
        ks.set_operand_copies(mode)
        ks.set_workspace(PTR if scratch else None, scratch)
        return ks.gemm_plan(dtype, kid, tA, tB, M, N, K, 1.0, PTR, (M if tA else K) + pad, PTR, (K if tB else N) + pad, 0.0, PTR, N)
    yield of
    ks.set_operand_copies(-1)
    ks.set_workspace(None)


def test_copies_leave_the_partitions_their_scratch(plan):
    """A count of K partitions that the scratch holds is not lowered by copies that take the scratch first."""
    sizes = [(2985, 1473, 14790, 0, 0, 128 << 20), (513, 3452, 14151, 0, 0, 128 << 20), (1024, 1024, 64001, 0, 1, 256 << 20)]
    rng = random.Random(5)
    while len(sizes) < 600:
        M, N, K = (int(2 ** rng.uniform(*r)) for r in ((8, 13), (8, 13), (10, 16)))
        if 1e10 <= 2.0 * M * N * K <= 2e12:
            sizes.append((M, N, K, rng.randint(0, 1), rng.randint(0, 1), rng.choice([32, 64, 128, 256]) << 20))
    split = 0
    for M, N, K, tA, tB, scratch in sizes:
        kid = plan(0, scratch, tA, tB, M, N, K)["kernel_id"]
        # the scratch at hand, and exactly what the member is said to use
        for size in (scratch, ks.workspace_bytes_needed(ks.BF16, kid, M, N, 1)):
            without, has = plan(0, size, tA, tB, M, N, K), plan(-1, size, tA, tB, M, N, K)
            assert has["split_k"] == without["split_k"], (M, N, K, tA, tB, size, without, has)
            split += without["split_k"] > 1
    assert split > 300
