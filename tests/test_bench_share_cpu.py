"""The bytes that a batched launch is counted with: those of the systems still
running, over every system whose hierarchy has the level."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench


def test_active_share():
    ns, cycles = [127, 127, 511, 1023], [2, 4, 6, 8]
    # all four have a level of 127 points (and of 63), the larger two one of 255
    assert bench.active_share("pre n=127", ns, cycles) == pytest.approx((2 + 4 + 6 + 8) / 32)
    assert bench.active_share("post_tile n=63", ns, cycles) == pytest.approx(20 / 32)
    assert bench.active_share("pre n=255", ns, cycles) == pytest.approx((6 + 8) / 16)
    assert bench.active_share("pre n=1023", ns, cycles) == 1.0
    assert bench.active_share("tail", ns, cycles) == pytest.approx(20 / 32)
    pts = [m * m for m in ns]
    assert bench.active_share("norm", ns, cycles) == pytest.approx(
        sum((c + 1) * p for c, p in zip(cycles, pts)) / (9 * sum(pts)))
