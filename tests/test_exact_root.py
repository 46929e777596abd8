"""The exact stabilizer away from equilibrium, on the CPU: its general search over
states 20-30% from equilibrium, against the oracle's bisection, and the
logarithm it uses there."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def test_no_state_far_from_equilibrium_gets_a_wrong_root(orc):
    """A rounding error e of the logarithms' sum moves a population by at most
    about e sqrt(f'_i sum_j f^eq_j / (1 + x_j)) (Cauchy-Schwarz on dh_i sum
    |dh_j| / sum dh_j^2 / f'_j), with 27 terms below 1e-11 even where some
    1 + x_j is 1e-10; a gamma off by 1e-2 moves it by 1e-5.  1e-9 lies between."""
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not present")
    odir = os.path.join(ROOT, "oracle")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "root")
        subprocess.run([CLANG, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", CSRC, "-I", odir, os.path.join(ROOT, "tests", "host", "exact_root_check.cpp"),
                        "-L", odir, "-lkbc_oracle", f"-Wl,-rpath,{odir}", "-lpthread", "-o", exe],
                       check=True, capture_output=True)
        r = subprocess.run([exe, "400000", "1e-9"], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr


def test_logarithm_for_any_argument():
    """Within 3e-16 (1 + |ln(1 + x)|): half an ulp of 1 + x (1.1e-16 in ln), one rounding
    each of 2 t, the quotient t and the result (below 1.1e-16 of 0.35 or of the
    result), k ln 2 within 2^-54 of itself, truncation below 2e-18."""
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not present")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "ln")
        subprocess.run([CLANG, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", CSRC, os.path.join(ROOT, "tests", "host", "log1p_any_check.cpp"), "-o", exe],
                       check=True, capture_output=True)
        r = subprocess.run([exe, "3e-16"], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
