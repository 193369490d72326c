"""Registers of the largest 16-bit tile on the register-staged path: what the compiler spills runs in every K-step."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_06795_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the device compiler")
@pytest.mark.parametrize("layout,most", [("false, false", 39), ("true, false", 14)])
def test_unsplit_256_x_256_tile(tmp_path, layout, most):
    """TN and NN, where the step that holds the end of K has one form: no more spills than with that form alone."""
    src = tmp_path / "one.hip"
    src.write_text('#include "gemm_bf16.hpp"\n'
                   "template __global__ void ks::gemm_bf16_kernel<16, 256, 256, 64, 128, 64, false, %s>(const ks::GemmParams);\n" % layout)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-I", CSRC, "-c", str(src), "-o",
                        str(tmp_path / "one.o")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    spills = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert spills and max(spills) <= most, spills
