"""The rules by which a box's launches are chosen, on the CPU (a host build of
kbc_internal.h): each test names the boxes for which another choice was measured to
be slower."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1507_02518_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not present")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    subprocess.run([CLANG, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", CSRC, os.path.join(ROOT, "tests", "host", "launch_rules.cpp"), "-o", exe],
                   check=True, capture_output=True)

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]

    return run


def test_curl_runs_fill_the_gpu_on_thin_boxes(rule):
    # a thread for every few nodes where planes are small
    for shape in ((1, 1, 4000000), (4, 4, 500000), (1, 1, 65536), (8, 8, 8192)):
        lz, runs = rule("curl", *shape)
        assert lz == 4 and runs * 4 >= shape[0] * shape[1] * shape[2], shape
    assert rule("curl", 512, 512, 512)[0] == 32


def test_stabilizer_statistics_take_few_rounds_of_workgroups(rule):
    assert rule("gamma", 1, 1, 1) == [1] and rule("gamma", 33, 17, 65) == [143]
    assert rule("gamma", 100, 100, 100) == [1024] and rule("gamma", 512, 512, 512) == [1024]
