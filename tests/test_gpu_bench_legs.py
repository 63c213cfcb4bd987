"""The benchmark's 1-D legs report no bandwidth reckoned from single steps: a
launch makes several steps per pass over the state."""
import pytest

pytestmark = pytest.mark.gpu


def test_1d_legs_report_no_step_bandwidth():
    import bench

    assert "achieved_GBs" not in bench.run_tube1d(n=1 << 16, steps=20)
    assert "achieved_GBs" not in bench.run_batch("fp32", steps=20, n_tubes=8)
