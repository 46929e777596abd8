"""Rows padded for the pair sweep cost memory that a box does without where it is not
there: an allocation limit between the two sizes (a hipMalloc of the test's own,
in a process of its own), and one below both."""
import os
import subprocess
import sys
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import ctypes, sys
import numpy as np
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import oracle as orc
from paper_1507_02518_amd import inputs, kbc
shape, nu = (100, 61, 60), 1e-2
u = inputs.smooth_random(shape, 0.04, seed=3)
try:
    b = kbc.Box(shape, nu)
except kbc.KbcError as e:
    print("refused", e.code)
    sys.exit(0)
with b:
    b.init_velocity(u)
    b.step(5)
    f = b.populations()
F = orc.run(orc.init_feq(u), orc.beta_from_nu(nu), 5)
print("runs", float(np.abs(f - F).max()) <= 1e-13)
"""


@pytest.mark.gpu
def test_box_is_made_without_padding_where_the_padded_one_does_not_fit():
    node = 27 * 8
    plain, padded = 100 * 61 * 60 * node, 112 * 61 * 60 * node
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "limit.so")
        subprocess.run(["gcc", "-O2", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host", "malloc_limit.c"),
                        "-ldl", "-o", so], check=True)

        def run(limit):
            env = dict(os.environ, KBC_TEST_MALLOC_LIMIT=str(limit), PYTHONPATH=ROOT)
            r = subprocess.run([sys.executable, "-c", CODE, so], env=env, cwd=ROOT, capture_output=True,
                               text=True, timeout=100)
            assert r.returncode == 0, r.stdout + r.stderr
            return r.stdout.strip().splitlines()[-1]

        assert run(2 * padded) == "runs True"
        # no allocation of the padded lattice, but of everything the box needs
        assert run((plain + padded) // 2) == "runs True"
        assert run(plain // 2) == "refused -2"       # KBC_ENOMEM
