"""Pricing of the step's roofline: a step of the table that this design does without one record per
instance, or without the SH rows, is priced by the bytes the design moves, so that no rate comes
out above what the memory reaches."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402

COUNTS = dict(N=1_000_000, n_vis=857_000.0, K=8.47e6, P=1920 * 1080, tiles=120 * 68)


def test_steps_done_otherwise_are_priced_by_their_own_bytes():
    N, n_vis, K, P, tiles = COUNTS.values()
    for step in ("S3 scan", "S4 duplicate", "S5 sort", "S6 ranges", "S9 preprocess backward"):
        own = sum(bench.algorithmic_bytes(s, N, n_vis, K, P, tiles) for s in bench.SURVEY_STEPS[step])
        assert bench.step_work(step, N, n_vis, K, P, tiles, 1.7e8, 8.2e7) == (own, 0.0)
    # the tiles' bounds are found from the tiles' lengths alone, whatever the instances
    assert bench.step_work("S6 ranges", N, n_vis, 10 * K, P, tiles, 0, 0)[0] == 16 * tiles


def test_the_other_steps_keep_the_tables_work():
    N, n_vis, K, P, tiles = COUNTS.values()
    for step in ("S2 preprocess", "S7 blend", "S8 blend backward"):
        assert bench.step_work(step, N, n_vis, K, P, tiles, 1.7e8, 8.2e7) == \
            bench.survey_work(step, N, K, P, tiles, 1.7e8, 8.2e7)
