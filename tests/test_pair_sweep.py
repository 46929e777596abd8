"""Two steps of a pull box in one sweep (k_pair): the plan and its index rules
on the CPU; on the GPU, the populations against the same box advanced by
single steps, bit for bit (the two take the same collision on the same
inputs), and against the oracle."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from paper_1507_02518_amd import inputs, kbc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")
F64, F32 = kbc.F64, kbc.F32_DEV

# shape, storage, variant: whole tiles; partial tiles on every axis in rows
# that are not padded (15 of 65 nodes); padded rows; the last tile one column
# and one row wide; the fewest planes per tile; FP32 at its smallest.
SHAPES = [((64, 64, 64), F64, kbc.S_DTQ), ((65, 63, 71), F64, kbc.S_DTQ),
          ((100, 61, 60), F64, kbc.S_D), ((113, 73, 48), F64, kbc.S_DT),
          ((112, 96, 33), F64, kbc.S_CDTQ), ((256, 192, 5), F64, kbc.S_DTQ),
          ((160, 160, 160), F32, kbc.S_DTQ), ((192, 101, 160), F32, kbc.S_DQ)]


def _host_check(d):
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("ROCm clang++ not present")
    exe = os.path.join(d, "pair")
    subprocess.run([clang, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", CSRC, os.path.join(ROOT, "tests", "host", "pair_check.cpp"), "-o", exe],
                   check=True)
    return exe


def test_plan_and_index_rules_on_the_host():
    with tempfile.TemporaryDirectory() as d:
        exe = _host_check(d)
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        # the GPU test's boxes take their steps in pairs
        for shape, dtype, variant in SHAPES:
            r = subprocess.run([exe, str(dtype), *map(str, shape), str(variant)],
                               capture_output=True, text=True, check=True)
            assert r.stdout.startswith("pairs"), (shape, dtype, variant, r.stdout)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dtype,variant", SHAPES)
def test_pairs_give_the_bits_of_single_steps(orc, shape, dtype, variant):
    print(f"pairs {shape} dtype={dtype} variant={variant}", flush=True)
    u = inputs.hit(shape, 2.0, 0.04, seed=sum(shape))
    nu, steps = 1e-3, 7
    with kbc.Box(shape, nu, dtype, variant=variant) as b:
        b.init_velocity(u)
        b.step(steps)           # three pairs and a single step
        f = b.populations()
        b.step(1)
        b.step(37)              # starts in the other buffer: a pair, graphs of 16, the rest
        t, g = b.t, b.populations()
    with kbc.Box(shape, nu, dtype, variant=variant) as b:
        b.init_velocity(u)
        for _ in range(steps):
            b.step(1)
        f1 = b.populations()
        for _ in range(38):
            b.step(1)
        g1 = b.populations()
    assert t == steps + 38
    assert np.array_equal(f, f1)
    assert np.array_equal(g, g1)
    if dtype == F64:
        # 1e-13 after a few steps: the bound of the ragged-box parity tests
        F = orc.run(orc.init_feq(u), orc.beta_from_nu(nu), steps, variant=variant)
        assert np.abs(f - F).max() <= 1e-13
