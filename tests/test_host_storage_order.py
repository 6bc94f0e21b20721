"""The storage order of the coefficients (AGCA_ELEM_SOA, csrc/kuhn.h): a build with the order that the
two-product passes do not read has to fail."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_13109_amd", "csrc")


@pytest.mark.parametrize("soa", [0, 1])
def test_two_product_passes(soa):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only", "-fsyntax-only", f"-DAGCA_ELEM_SOA={soa}",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "k_smooth2.hip")],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == (soa == 0), r.stderr
    assert soa == 0 or "six coefficients as one run" in r.stderr
