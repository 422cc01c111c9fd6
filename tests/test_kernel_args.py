"""The products and reductions of the solve phase are launched in chains, where a
launch's host time counts: none of their kernels takes the compiler's hidden
arguments (256 bytes with each launch, for gridDim and the like)."""
import os
import re
import subprocess

import pytest

from paper_1008_1700_amd import build as B


@pytest.mark.parametrize("src,kernels", [("k_gemv.hip", ("k_gemv", "k_gemv_n", "k_gemv_w", "k_gemv_mf32", "k_tipmv", "k_tipmv_c")),
                                         ("k_vec.hip", ("k_reduce2", "k_reduce2_part")),
                                         ("k_ilu.hip", ("k_ilu_solve_lds",)), ("k_panel.hip", ("k_panel",))])
def test_no_hidden_arguments(src, kernels, tmp_path):
    out = tmp_path / "k.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", str(out)], check=True,
                   capture_output=True)
    seen = set()
    for entry in re.split(r"\n  - (?=\.)", out.read_text().split("amdhsa.kernels:")[1]):
        name = re.search(r"\.name:\s+_ZN4ddps(?:12_GLOBAL__N_1)?\d+(k_\w+?)(?:I[dfL]|E)", entry)
        if name and name.group(1) in kernels:
            seen.add(name.group(1))
            assert "hidden_" not in entry, name.group(0)
    assert seen == set(kernels)
