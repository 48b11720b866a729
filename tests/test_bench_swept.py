"""The roofline object's bytes count the nodes that bottom-up steps pass over."""

import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


def test_swept_nodes_are_counted():
    assert bench.algorithmic_bytes(0, 0, 0, 64, swept=10) == 10 * (8 + 4)
    assert bench.algorithmic_bytes(0, 0, 0, 256, trial=False, swept=3) == 3 * (32 + 4)
    assert bench.algorithmic_bytes(5, 6, 7, 256, trial=False, swept=1) == \
        bench.algorithmic_bytes(5, 6, 7, 256, trial=False) + 36
