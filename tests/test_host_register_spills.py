"""Registers of kernels whose speed hangs on a few of them: what the compiler spills runs in every K-step, and one register
over a budget costs a resident work-group."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_06795_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the device compiler")


def resources(tmp_path, header, kernel):
    src = tmp_path / "one.hip"
    src.write_text('#include "%s"\ntemplate __global__ void ks::%s(const ks::GemmParams);\n' % (header, kernel))
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-I", CSRC, "-c", str(src), "-o",
                        str(tmp_path / "one.o")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    spills, waves = (re.findall(what + r": (\d+)", r.stderr) for what in ("VGPRs Spill", r"Occupancy \[waves/SIMD\]"))
    assert len(spills) == 1 and len(waves) == 1, r.stderr[-2000:]
    return int(spills[0]), int(waves[0])


@pytest.mark.parametrize("layout,most", [("false, false", 39), ("true, false", 14)])
def test_unsplit_256_x_256_tile(tmp_path, layout, most):
    """TN and NN, where the step that holds the end of K has one form: no more spills than with that form alone."""
    assert resources(tmp_path, "gemm_bf16.hpp", "gemm_bf16_kernel<16, 256, 256, 64, 128, 64, false, %s>" % layout)[0] <= most


@pytest.mark.parametrize("tile,layout", [("64, 64, 32", "true, false"), ("64, 64, 32", "false, true"), ("64, 64, 32", "true, true"),
                                         ("32, 32, 16", "true, true")])
def test_fp32_units_form_on_16_wide_fragments(tmp_path, tile, layout):
    """Sixteen waves of 64 x 64 hold two work-groups a compute unit, 32 x 32 x 16 eight: eight waves per SIMD, no spills."""
    assert resources(tmp_path, "gemm_f32.hpp", "gemm_f32_kernel<1, %s, 16, 16, false, %s, 1, 1, false, false>" % (tile, layout)) == (0, 8)


@pytest.mark.parametrize("balanced", ["false", "true"])
@pytest.mark.parametrize("layout", ["false, false", "false, true", "true, false", "true, true"])
def test_fp32_parts_on_128_x_128_tiles(tmp_path, layout, balanced):
    """Two work-groups of eight waves a compute unit take 128 registers a wave, 64 of them accumulators: none over that, in the
    balanced form's loop over tiles neither."""
    assert resources(tmp_path, "gemm_f32_parts.hpp", "gemm_f32_parts_kernel<128, 128, 64, 32, false, %s, 1, %s>" % (layout, balanced)) == (0, 4)
