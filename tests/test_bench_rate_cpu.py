"""The bench's speed-ups compare a batch with the plain form over the plain form's steps."""
import bench


def test_rate_over_the_first_steps():
    run = {"solved": [100, 100, 50, 0], "lat": [0.5, 0.5, 1.0, 8.0], "value": 25.0}
    assert bench.rate_over(run, 2) == 200.0
    assert bench.rate_over(run, 3) == 125.0
    assert bench.rate_over(run, 4) == 25.0
    assert bench.rate_over(run, 9) == 25.0  # no more steps than there were
