"""CPU checks of the bench's byte counts of the stages that walk neighbour lists."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


@pytest.mark.parametrize("K,R", [(8, 10), (16, 10), (32, 0)])
def test_empty_places_are_not_charged(K, R):
    import bench
    full, one = bench.list_bytes(K, K, 32.0, R), bench.list_bytes(K, 1.0, 0.0, R)
    # full lists: every id, kernel value, pose and psi; a list of the particle alone: the ids and one of each
    assert full["svgd"] == 56.0 + 64.0 * K and one["svgd"] == 56.0 + 4 * K + 60.0
    assert full["posterior"] == 20.0 + R * (12.0 * K + 4) and one["posterior"] == 20.0 + R * (4.0 * K + 12)
    assert full["refresh"] == 28.0 + 40.0 * K + 32.0 * 32 and one["refresh"] == 28.0 + 12.0 * K + 28.0
    once = bench.compulsory_list_bytes(K, K, R), bench.compulsory_list_bytes(K, 1.0, R)
    assert once[0]["svgd"] == 8.0 * K + 96 and once[1]["svgd"] == 4.0 * K + 100
    assert once[0]["posterior"] == 36.0 + R * (8.0 * K + 8) and once[1]["posterior"] == 36.0 + R * (4.0 * K + 12)


def test_mean_lengths():
    import numpy as np

    import bench

    class F:
        def debug_get(self, name):
            return {"cnt": np.array([1, 1, 4, 6]), "head": np.array([0, 0, 0, 3]), "end": np.array([3, 3, 3, 60])}[name]
    assert bench.list_lengths(F(), dict(window_c=32)) == (3.0, (2 + 2 + 2 + 32) / 4)
