"""Where a selecting call takes the K-slices form of the 16-bit products (ks_launch_plan_t::path 16 + tile): one round of work-groups,
by direct-to-LDS loads (tiles 0 to 9) on aligned operands with whole K-steps of 64, through registers (10 to 18) on others, and
never for a named member, forced partitions, a caller's own tree, batches or fp32.  No GPU: ks_gemm_plan reads sizes and addresses
only."""
import ctypes
import re
import shutil
import subprocess

import pytest

import paper_2003_06795_amd.binding as ks
from paper_2003_06795_amd import build as lib_build

TILES = [tile[:2] for tile in lib_build.slice_tiles()]
PTR = 1 << 20


@pytest.fixture()
def planner():
    L = ks.lib()
    assert L.ks_set_workspace(ctypes.c_void_p(1 << 21), ctypes.c_size_t(256 << 20)) == 0

    def plan(dtype, kid, tA, tB, M, N, K, batch=1, lda=None, ldb=None, a=PTR):
        return ks.gemm_plan(dtype, kid, tA, tB, M, N, K, 1.0, a, lda or (M if tA else K), PTR, ldb or (K if tB else N), 0.0, PTR, N,
                            batch, M * K, K * N, M * N)
    yield plan
    L.ks_set_workspace(None, 0)


@pytest.mark.parametrize("odd", [0, 1])
def test_the_form_is_one_round_of_its_tiles(planner, odd):
    seen = set()
    for tA in (0, 1):
        for tB in (0, 1):
            for M in (8, 64, 256, 1024, 3368, 4096, 8192, 16384):
                for N in (8, 40, 64, 152, 512, 1024, 12000):
                    for K in (192, 256, 448, 512, 1024, 2048, 3008, 4096, 8192):
                        for dtype in (ks.BF16, ks.F16):
                            got = planner(dtype, -1, tA, tB, M - odd, N - odd, K - odd)
                            if got["path"] < 16:
                                continue
                            bm, bn = TILES[got["path"] - 16]
                            tiles = -(-(M - odd) // bm) * -(-(N - odd) // bn)
                            assert K >= (256 if odd else 512) and (got["path"] >= 26) == bool(odd)
                            assert tiles <= 256 and got["workgroups"] == tiles and got["split_k"] == 1, got
                            assert got["kernel_id"] == ks.select(dtype, M - odd, N - odd, K - odd, 1, tA, tB)
                            assert not (got["tail_split"] or got["k_remainder"] or got["operand_copies"] or got["balanced_groups"])
                            seen.add(got["path"] - 16)
    assert seen == (set(range(10, 19)) if odd else set(range(10)))


def test_calls_that_do_not_take_it(planner):
    size = (0, 1, 512, 512, 2048)
    assert planner(ks.BF16, -1, *size)["path"] == 16 + 3
    assert planner(ks.BF16, ks.select(ks.BF16, 512, 512, 2048, 1, 0, 1), *size)["path"] < 16
    assert planner(ks.F32, -1, *size)["path"] < 16
    assert planner(ks.BF16, -1, *size, batch=2)["path"] < 16
    assert planner(ks.BF16, -1, *size, a=PTR + 2)["path"] >= 26
    assert planner(ks.BF16, -1, *size, lda=2052)["path"] >= 26
    assert planner(ks.BF16, -1, 0, 1, 512, 512, 2080)["path"] >= 26
    assert planner(ks.BF16, -1, 0, 0, 512, 516, 2048)["path"] >= 26         # rows of B end inside sixteen bytes
    assert planner(ks.BF16, -1, 0, 1, 512, 507, 2048)["path"] == 16 + 3     # columns of C may end anywhere
    assert planner(ks.BF16, -1, 0, 0, 3000, 6, 2001)["path"] < 16           # rows of six elements: B from further back does not work
    assert planner(ks.BF16, -1, 0, 0, 3000, 6, 2001, ldb=7)["path"] >= 26
    assert planner(ks.BF16, -1, 1, 0, 1024, 1024, 5001)["path"] < 16        # copies of the operands pay
    assert planner(ks.BF16, -1, 0, 0, 8001, 9, 4195)["path"] < 16           # 2^25 entries of A
    # that the member is faster at (time of the form over its): rows between lines 1.21, what is in flight of 50 MiB 1.08, the
    # largest tile for the 64 x 64 x 128 member 1.17
    assert planner(ks.BF16, -1, 0, 1, 1984, 448, 3584, lda=3592, ldb=3592)["path"] < 16
    assert planner(ks.BF16, -1, 0, 1, 1984, 448, 3584)["path"] == 16 + 8
    assert planner(ks.BF16, -1, 0, 1, 2944, 52, 8960)["path"] < 16
    assert planner(ks.BF16, -1, 1, 1, 2816, 212, 7808)["path"] < 16
    ks.set_split_partitions(2)
    try:
        assert planner(ks.BF16, -1, *size)["path"] < 16
    finally:
        ks.set_split_partitions(0)
    ks.set_operand_copies(1)                                                 # copies wherever they can be made: by the member
    try:
        got = planner(ks.BF16, -1, 0, 1, 975, 675, 3392, lda=3396)
        assert got["path"] < 16 and got["operand_copies"] == 1
        got = planner(ks.BF16, -1, 0, 1, 975, 675, 3365, a=PTR + 2)
        assert got["path"] < 16 and got["operand_copies"] == 3
        assert planner(ks.BF16, -1, *size)["path"] == 16 + 3                 # none to be made
        for mode in (0, -1):
            ks.set_operand_copies(mode)
            assert planner(ks.BF16, -1, 0, 1, 975, 675, 3392, lda=3396)["path"] >= 26
    finally:
        ks.set_operand_copies(-1)
    ks.set_fast_path(False)
    try:
        assert planner(ks.BF16, -1, *size)["path"] < 16
    finally:
        ks.set_fast_path(True)
    tree = ks.get_selector(ks.BF16)
    ks.set_selector(ks.BF16, tree)
    try:
        assert planner(ks.BF16, -1, *size)["path"] < 16
    finally:
        ks.set_selector(ks.BF16, [])
    ks.lib().ks_set_workspace(None, 0)                                       # it needs no scratch
    assert planner(ks.BF16, -1, *size)["path"] == 16 + 3


def assembly(tmp_path, kernel):
    src, asm = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "gemm_bf16_slices.hpp"\ntemplate __global__ void ks::%s;\n' % kernel)
    subprocess.run([lib_build.HIPCC] + lib_build.HIP_FLAGS + ["-I", lib_build.CSRC, "--cuda-device-only", "-S", str(src), "-o",
                                                              str(asm)], check=True, capture_output=True)
    return asm.read_text().splitlines()


@pytest.mark.skipif(shutil.which(lib_build.HIPCC) is None, reason="needs the device compiler")
@pytest.mark.parametrize("tile,layout", [("16, 16, 64, 8, 4", "true, true"), ("32, 32, 64, 8, 2", "false, true"),
                                         ("64, 64, 64, 4, 2", "true, false"), ("64, 32, 64, 4, 3", "false, false")])
def test_a_stage_is_refilled_behind_its_reads(tmp_path, tile, layout):
    """The direct-to-LDS loads of the K loop overwrite the stage that the step before has read: between the wait that opens
    a step and its loads the code waits for the LDS reads too."""
    lines = assembly(tmp_path, "gemm_bf16_slices_kernel<%s, %s, false>(const ks::HotPointers, const ks::HotInts, const ks::HotInts, const "
                               "ks::GemmParams, const int)" % (tile, layout))
    step, waited, refills = False, False, 0
    for line in lines:
        if re.search(r"s_waitcnt vmcnt\(\d+\)", line):
            step, waited = True, "lgkmcnt(0)" in line
        elif "s_waitcnt" in line and "lgkmcnt(0)" in line:
            waited = True
        elif "ds_read" in line:
            waited = False
        elif "global_load_lds" in line and step:
            refills += 1
            assert waited, line
    assert refills > 0


@pytest.mark.skipif(shutil.which(lib_build.HIPCC) is None, reason="needs the device compiler")
@pytest.mark.parametrize("bm,bn,bk,rest,layout", [(16, 16, 64, "16, 4", "false, false"), (16, 16, 64, "16, 4", "true, true"),
                                                  (32, 16, 64, "8, 3", "false, true"), (64, 64, 32, "8, 3", "true, false")])
def test_lanes_read_a_step_behind_all_writes_of_it(tmp_path, bm, bn, bk, rest, layout):
    """The lanes of a wave read from LDS what others of them have written, where the compiler looks at one lane's addresses: no
    read stands between the writes of a K-step (nor of the sums, one a fragment, at the end)."""
    lines = assembly(tmp_path, "gemm_bf16_slices_staged_kernel<%d, %d, %d, %s, %s, false>(const ks::GemmParams)" % (bm, bn, bk, rest, layout))
    runs, run = [], 0
    for line in lines + [".L"]:
        if "ds_write" in line:
            run += 1
        elif "ds_read" in line or line.startswith(".L"):
            runs += [run] if run else []
            run = 0
    step, sums = (bm + bn) * bk * 2 // 1024, bm * bn // 256
    runs.remove(sums)
    assert len(runs) > 1 and all(n % step == 0 for n in runs), runs
