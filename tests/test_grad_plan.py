"""How the gradient sums are split over the GPU: small boxes must not be left to a
few workgroups that march through many planes, thin boxes not to tiles whose lanes
are mostly empty; on the GPU, the sums at the edges of that rule against the oracle."""
import os
import subprocess
import tempfile

import pytest

from oracle import statistics as ost
from paper_1507_02518_amd import inputs, kbc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def test_small_and_thin_boxes_fill_the_gpu():
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not present")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "gp")
        subprocess.run([CLANG, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", CSRC, os.path.join(ROOT, "tests", "host", "grad_plan_check.cpp"), "-o", exe],
                       check=True, capture_output=True)

        def plan(*shape):
            r = subprocess.run([exe, *map(str, shape)], capture_output=True, text=True, check=True)
            return tuple(int(v) for v in r.stdout.split())

        # one node per thread: small, or under 0.4 of the lanes filled
        for shape in ((32, 32, 32), (64, 64, 64), (33, 17, 65), (1, 1, 4000000), (4, 4, 500000),
                      (4, 512, 512), (8, 1024, 1024), (1, 2147483647, 1)):
            assert plan(*shape)[0] == 0, shape
        # tiles, in marches short enough for a workgroup on most CUs
        for shape in ((65, 65, 64), (80, 80, 80), (131, 97, 61), (128, 128, 128), (16, 400, 400)):
            lz, items = plan(*shape)
            assert lz in (8, 16) and items >= 200, (shape, lz, items)
        assert plan(200, 200, 200)[0] == 16 and plan(512, 512, 512)[0] == 16


@pytest.mark.gpu
@pytest.mark.parametrize("order", [2, 8])
@pytest.mark.parametrize("shape", [(65, 65, 64), (300, 5, 200), (31, 300, 42), (256, 256, 130),
                                   (3, 400, 300), (600, 1, 500), (64, 64, 64), (3, 1, 1), (5, 1, 60001)])
def test_gradient_statistics_at_the_edges_of_the_plan(shape, order):
    print(f"gradients {shape} order={order}", flush=True)
    with kbc.Box(shape, 2e-2) as b:
        b.init_velocity(inputs.smooth_random(shape, 0.05, seed=9))
        b.step(2)
        got = b.statistics(order)
        _, u = b.moments()
    ref = ost.statistics(u, 2e-2, order)
    for key in ("k", "omega", "epsilon", "div2"):
        assert got[key] == pytest.approx(ref[key], rel=1e-12, abs=1e-28), key
    for n in range(2, 7):
        # odd moments cancel: their rounding is that of the terms
        scale = ref["dudx_moments"][2] ** (n / 2)
        assert got["dudx_moments"][n] == pytest.approx(ref["dudx_moments"][n], rel=1e-11,
                                                       abs=1e-11 * scale + 1e-60), n
