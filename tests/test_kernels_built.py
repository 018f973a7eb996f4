"""The kernels in the shared library, by the host stubs it defines: none that the
dispatch cannot reach."""
import os
import re
import shutil
import subprocess

import pytest

NEVER = [
    # rows of 768 FP64 values are split, so the stride of a whole one serves FP32 alone
    r"k_sweep_rows<double, 772,",
    # a sweep starts from a zero correction in FP32 alone
    r"k_sweep_rows<double, \d+, \d, [12]>",
    r"k_sweep_tile<double, \d+, \d, [12]>",
    # neighbours of rows that do not fill a run of lanes: by lane in FP32, loaded in FP64
    r"k_(colour_pair_gen|colour_pair_split)<double, \d, 2>", r"k_residual_pair_gen<double, 2>",
    r"k_(colour_pair_gen|colour_pair_split)<float, \d, 0>", r"k_residual_pair_gen<float, 0>",
]


@pytest.mark.skipif(shutil.which("nm") is None, reason="nm is not installed")
def test_no_unreachable_kernel():
    from paper_1904_03808_amd import build
    if not os.path.exists(build.LIB):
        build.build_library()
    out = subprocess.run(["nm", "-C", build.LIB], capture_output=True, text=True, check=True).stdout
    stubs = [line for line in out.splitlines() if "__device_stub__" in line]
    assert any("k_sweep_rows<float, 772," in s for s in stubs)
    found = [s for s in stubs for pat in NEVER if re.search(pat, s)]
    assert not found, found[:5]
