"""The committed rocprofv3 summary that the bench line's traffic comes from: the pair
of steps of the headline box."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_headline_pair_traffic_is_its_bytes_and_the_halo():
    """Writes once, reads once and the tiles' halo: 18 x 14 nodes read for 16 x 12 stored
    and two planes more per march bound the reads by 1.35 of the algorithmic half."""
    traffic = bench.read_counters(bench.PAIR_COUNTERS, bench.PAIR_SOURCES)
    if traffic is None:
        pytest.skip("pair counters taken on other kernel sources (profiles need a new run)")
    algorithmic = 432 * bench.N ** 3
    assert 0.98 * algorithmic < traffic < (1.0 + 0.35 / 2) * algorithmic
