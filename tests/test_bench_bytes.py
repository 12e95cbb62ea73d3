"""Bytes and launches the benchmark states for a run, from the steps per pass the
library reports (no GPU)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench


class Grid:
    def __init__(self, steps_per_pass):
        self.steps_per_pass = steps_per_pass


@pytest.mark.parametrize("per_pass,steps,launches", [(1, 100, 100), (2, 100, 50), (2, 101, 51),
                                                     (4, 100, 25), (4, 7, 4), (2, 1, 1)])
def test_launches_of_a_run(per_pass, steps, launches):
    assert bench.launches(Grid(per_pass), steps) == launches
    assert bench.lup_bytes(Grid(per_pass), steps, 19, 4) == pytest.approx(152 * launches / steps)


def test_sources_of_profiled_kernels_exist():
    assert all(len(bench.kernel_hash(k)) == 16 for k in bench.SOURCES)
