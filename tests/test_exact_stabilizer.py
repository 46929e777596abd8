"""The exact stabilizer's single-pass root search: its wider logarithm
polynomials on the CPU, and on the GPU one collision of states at increasing
distance from equilibrium against the oracle's bisection, so that each
polynomial and the general search behind them are taken."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from paper_1507_02518_amd import inputs, kbc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")


def test_wide_log1p_polynomials_host_check():
    """Within 5e-16 relative (truncation below 8e-17, the rest is the rounding
    of a Horner scheme whose inner terms are scaled by |x| <= 1/4)."""
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("ROCm clang++ not present")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "lg")
        subprocess.run([clang, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host", "log1p_wide_check.cpp"), "-o", exe],
                       check=True)
        r = subprocess.run([exe, "5e-16"], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr


# Perturbations of the equilibrium with |x_i| of the order of the amplitude:
# below 1/16 in every wave, below 1/8, below 1/4 and beyond.  Bounds: those of
# the host build of the collision against the oracle (5e-15 near equilibrium,
# 2e-13 for 10-30% perturbations).
@pytest.mark.gpu
@pytest.mark.parametrize("amp,tol", [(1e-4, 5e-15), (0.01, 5e-15), (0.03, 2e-13), (0.06, 2e-13),
                                     (0.2, 2e-13)])
@pytest.mark.parametrize("streaming", [kbc.PULL, kbc.AA])
@pytest.mark.parametrize("shape", [(128, 4, 3), (33, 5, 3)])
def test_single_pass_root_against_the_oracle(orc, shape, streaming, amp, tol):
    print(f"exact root {shape} streaming={streaming} amp={amp}", flush=True)
    u = inputs.smooth_random(shape, 0.05, seed=7)
    F = orc.init_feq(u)
    F = F * (1.0 + amp * np.random.default_rng(11).standard_normal(F.shape).clip(-2.5, 2.5))
    nu = 1e-3
    for variant in (kbc.S_DTQ, kbc.S_CDT):
        G = orc.run(F, orc.beta_from_nu(nu), 1, variant=variant, exact=True)
        with kbc.Box(shape, nu, variant=variant, streaming=streaming, gamma="exact") as b:
            b.set_populations(F)
            b.step(1)
            f = b.populations()
        assert np.abs(f - G).max() <= tol, (variant, np.abs(f - G).max())
