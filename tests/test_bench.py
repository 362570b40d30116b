"""Figures of the benchmark that are computed on the host."""

import bench


def test_one_slow_call_does_not_move_a_stage():
    """The first launch of a kernel takes milliseconds; the stage times are medians."""
    rows = [[0.004, 0.040, 0.019, 0.010]] * 19 + [[0.004, 1.700, 1.800, 0.010]]
    assert bench.stage_medians(rows, ["fold", "score", "value", "combine"]) == {"fold": 4.0, "score": 40.0, "value": 19.0, "combine": 10.0}
