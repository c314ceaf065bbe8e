"""The P2G launches behind bench.py's roofline figure, counted by hand from when
a run bins (every R sub-steps of the run, and at the start of every checkpoint
segment), and the bytes of their mean launch.  CPU only."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_launches_by_hand():
    # forward run: the launches at 0, 8 and 16 of 20 bin first; 0 alone without a binning interval
    assert bench.p2g_launches(20, 8) == (3, 17, 0)
    assert bench.p2g_launches(20, 0) == (1, 19, 0)
    # 500 sub-steps in segments of 50, binned every 32, the last 5 segments
    # recorded: all segments once as recorded ones, 25 binnings (10 starts, the 16
    # multiples of 32, of which 0 is a start); 250 unrecorded ones before, 12
    # binnings (5 starts, 8 multiples); the traced pass has 37 and 713
    assert bench.p2g_launches(500, 32, 50, 5) == (37, 713, 475)
    # every segment recorded: nothing is run twice; a ragged last segment
    assert bench.p2g_launches(500, 32, 50, 10) == (25, 475, 475)
    assert bench.p2g_launches(45, 8, 20, 1) == (7 + 6, 72, 38)
    # launches that never join
    assert bench.p2g_launches(500, 32, 50, 5, joins=False) == (750, 0, 0)
    assert bench.p2g_launches(20, 8, joins=False) == (20, 0, 0)


def test_mean_bytes_by_hand():
    # 3D FP32: 132 B a particle and 16 B a node by itself; joined x and G read and
    # written (96 B), a recorded one v and C as well (48 B), 28 B a node
    plain, joined, recorded = 1000 * 132 + 170 * 16, 1000 * 96 + 170 * 28, 1000 * 48
    assert bench.algorithmic_bytes_p2g_mean(1000, 170, (3, 0, 0)) == pytest.approx(plain)
    assert bench.algorithmic_bytes_p2g_mean(1000, 170, (3, 17, 0)) == pytest.approx((3 * plain + 17 * joined) / 20)
    assert bench.algorithmic_bytes_p2g_mean(1000, 170, (3, 17, 5)) == \
        pytest.approx((3 * plain + 17 * joined + 5 * recorded) / 20)
