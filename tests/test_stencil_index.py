"""The periodic neighbours of the gradient statistics on the CPU, up to the
longest axis a box may have."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def test_stencil_neighbours_on_every_axis_length():
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not present")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "per")
        subprocess.run([CLANG, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", CSRC, os.path.join(ROOT, "tests", "host", "periodic_check.cpp"), "-o", exe],
                       check=True, capture_output=True)
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
