"""Order of the LDS traffic of the sub-tile kernel (k_panel.hip), read from the
IR the compiler makes of it for gfx950.  Each product of its inversions reads
what other lanes stored for it (in FP32 across the lanes of a wave, in the last
step across waves), so a barrier of the wave or the workgroup, with its fences,
stands between any two of them."""
import os
import re
import subprocess

import pytest

from paper_1008_1700_amd import build as B


@pytest.fixture(scope="module")
def panel_ir(tmp_path_factory):
    out = tmp_path_factory.mktemp("ir") / "k_panel.ll"
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", "-emit-llvm",
                    os.path.join(B.CSRC, "k_panel.hip"), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


@pytest.mark.parametrize("kernel,product", [("k_panelId", "mfma.f64"), ("k_panelIf", "mfma.f32")])
def test_a_barrier_between_dependent_products(panel_ir, kernel, product):
    body = re.search(r"^define [^\n]*%s.*?^}" % kernel, panel_ir, re.S | re.M).group(0)
    runs, fenced = [0], False
    for line in body.splitlines():
        if "call" in line and product in line:
            runs[-1] += 1
        elif re.search(r"fence syncscope\(\"(wavefront|workgroup)\"\) release", line):
            fenced = True
        elif "barrier()" in line:
            assert fenced
            fenced = False
            runs.append(0)
    # 16 x 16 inner product and result, then 32 x 32 ones, four k per instruction
    assert [n for n in runs if n] == [4, 4, 8, 8]
