"""Waves per SIMD that a kernel's registers and LDS leave, as the compiler
reports them (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2112_07552_amd import build_lib


@pytest.mark.parametrize("source,kernel,waves", [("bsr.hip", "bsr_product_kernel", 8)])
def test_waves_per_simd(source, kernel, waves, tmp_path):
    if shutil.which(build_lib.HIPCC) is None:
        pytest.skip("no hipcc")
    r = subprocess.run([build_lib.HIPCC, *build_lib.FLAGS, "--cuda-device-only", "-c",
                        "-Rpass-analysis=kernel-resource-usage",
                        os.path.join(build_lib.CSRC, source), "-o", str(tmp_path / "k.o")],
                       capture_output=True, text=True, check=True)
    names = re.split(r"Function Name: ", r.stderr)[1:]
    found = [n for n in names if kernel in n.split()[0]]
    assert found
    for n in found:
        assert int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", n)[1]) == waves
        assert int(re.search(r"VGPRs Spill: (\d+)", n)[1]) == 0
