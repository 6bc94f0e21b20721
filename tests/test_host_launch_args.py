"""Size of the one-workgroup cycle's argument block (CoarseCycle, csrc/internal.h), which is copied
in every launch: with 1.8 KB the launch call of a new hierarchy's first cycle took up to 80 us
on the host, with 1 KB and less 7.  Bound: 768 bytes, FP64."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_13109_amd", "csrc")
ROCM = "/opt/rocm/include"


def test_coarse_cycle_arguments_are_small(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(os.path.join(ROCM, "hip")):
        pytest.skip("no host C++ compiler or HIP headers")
    src = tmp_path / "size.cpp"
    src.write_text('#include <cstdio>\n#include "internal.h"\n'
                   'int main() { std::printf("%zu %zu\\n", sizeof(agca::CoarseCycle<double>), sizeof(agca::CoarseCycle<float>)); }\n')
    exe = str(tmp_path / "size")
    inc = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")
    subprocess.run([gxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I", inc, "-I", CSRC, str(src), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    assert max(int(v) for v in out) <= 768
