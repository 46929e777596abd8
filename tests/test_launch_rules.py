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


F64, F32, DTQ, CDTQ = 0, 1, 3, 7


def test_pairs_on_planes_only_where_rows_are_aligned(rule):
    # 4 GiB and more: single steps are faster on these
    for shape in ((276, 276, 276), (290, 290, 290), (310, 310, 310), (350, 350, 350), (281, 500, 200),
                  (301, 300, 300)):
        assert rule("pair", F64, DTQ, *shape) == [0] and rule("pair", F64, CDTQ, *shape) == [0], shape
    for shape in ((384, 384, 384), (512, 512, 512), (512, 512, 160), (1024, 256, 160)):
        assert rule("pair", F32, DTQ, *shape) == [0], shape
    # and pairs on these
    for shape in ((280, 280, 280), (320, 320, 320), (512, 512, 512), (1000, 200, 200), (301, 301, 301)):
        assert rule("pair", F64, DTQ, *shape) == [1], shape
    for shape in ((352, 352, 352), (256, 512, 320), (96, 700, 700)):
        assert rule("pair", F32, DTQ, *shape) == [1], shape
    # below 4 GiB the rows' alignment does not matter
    for shape in ((256, 256, 256), (250, 250, 250), (97, 256, 256), (64, 64, 64)):
        assert rule("pair", F64, DTQ, *shape) == [1], shape


def test_no_fp32_pairs_in_the_last_level_cache(rule):
    # single steps through the caches are as fast or faster
    for shape in ((96, 96, 128), (256, 240, 12), (256, 480, 6), (512, 240, 6), (256, 480, 8)):
        assert rule("pair", F32, DTQ, *shape) == [0], shape
    for shape in ((160, 160, 160), (512, 512, 16), (96, 200, 200)):
        assert rule("pair", F32, DTQ, *shape) == [1], shape


def test_in_place_planes_that_share_cache_sets_store_past_the_caches(rule):
    for shape in ((128, 128, 128), (512, 64, 64), (64, 128, 256), (256, 256, 64)):
        assert rule("aa", F64, *shape) == [0], shape
    for shape in ((512, 64, 128), (256, 128, 128)):
        assert rule("aa", F32, *shape) == [0], shape
    # through them: other planes above the last-level cache, and those within it
    for shape in ((127, 127, 127), (160, 128, 128), (192, 128, 128), (200, 200, 200), (128, 128, 64),
                  (100, 100, 100)):
        assert rule("aa", F64, *shape) == [1], shape
    assert rule("aa", F32, 128, 128, 128) == [1] and rule("aa", F32, 256, 256, 128) == [1]


def test_in_place_fp64_boxes_little_above_the_l2s_store_past_the_caches(rule):
    assert rule("aa", F64, 56, 56, 56) == [0] and rule("aa", F64, 60, 60, 60) == [0]
    assert rule("aa", F64, 64, 64, 64) == [1] and rule("aa", F32, 72, 72, 72) == [1]
