"""The benchmark's figures that need no GPU."""
import bench


def test_steps_per_timed_launch_of_mixed_lengths():
    """1024^3, 2555 steps with a record every 50: 52 record passes of four
    steps and 510 timed launches of four and five."""
    per = bench.timed_steps_per_launch(2555, 52, 4, 0, 510)
    assert 4.0 < per < 5.0
    assert per * 510 + 52 * 4 == 2555
