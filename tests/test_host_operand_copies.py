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


def test_the_plan_reports_copies(plan):
    """A call that writes the scratch says so, also in one partition: beside split_k, tail_split stands operand_copies."""
    size = (0, 0, 4096, 4000, 4100)
    both = plan(-1, 256 << 20, *size, kid=45)
    assert (both["operand_copies"], both["split_k"], both["path"], both["vector_loads"]) == (3, 1, 0, 0)
    assert plan(0, 256 << 20, *size, kid=45)["operand_copies"] == 0
    assert plan(-1, 0, *size, kid=45)["operand_copies"] == 0                       # no scratch
    assert plan(-1, 32 << 20, *size, kid=45)["operand_copies"] == 0                # too little
    assert plan(1, 256 << 20, *size, kid=13)["operand_copies"] == 0                # split_k == 1: never the registered scratch
    assert plan(-1, 256 << 20, *size, kid=-1, dtype=ks.F32)["operand_copies"] == 0
    # one operand: whole K-steps, and only the rows of one are no multiple of eight
    def rows(lda, ldb):
        return ks.gemm_plan(ks.BF16, 45, 0, 1, 4096, 4000, 4096, 1.0, PTR, lda, PTR, ldb, 0.0, PTR, 4000)
    ks.set_operand_copies(-1)
    ks.set_workspace(PTR, 256 << 20)
    assert [rows(4096 + a, 4096 + b)["operand_copies"] for a, b in ((0, 0), (3, 0), (0, 3), (8, 8))] == [0, 1, 2, 0]
    # sixteen-byte accesses are legal, K is no whole number of half K-steps: what the operands admit is still reported
    got = ks.gemm_plan(ks.BF16, 45, 0, 1, 2048, 2048, 8168, 1.0, PTR, 8168, PTR, 8168, 0.0, PTR, 2048)
    assert (got["operand_copies"], got["vector_loads"], got["k_remainder"]) == (3, 1, 0)
