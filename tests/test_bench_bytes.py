"""The benchmark's byte count of a profiled run (no GPU)."""

import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


# stage launches by stage; fields moved per cell of the whole run
@pytest.mark.parametrize("n_stage,background,fields", [
    ([20, 20, 20, 20], False, 20 * 72),
    ([20, 20, 20, 20], True, 20 * 88),
    ([0, 20, 0, 20], False, 20 * 42),            # two stages per launch
    ([1, 21, 1, 21], False, 20 * 42 + 72),       # an odd number of steps: the last by single stages
    ([1, 1, 1, 1], False, 72),
])
def test_bytes_follow_the_launches(n_stage, background, fields):
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    assert bench.stage_accesses(n_stage, background) == fields
