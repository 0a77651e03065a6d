"""The benchmark's adjoint/forward ratios say which forward they are over (no GPU)."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_adjoint_ratio_over_each_forward():
    import bench
    # 100 steps back in 1500 ms; single steps of 5 ms, a timed run at 3.75 ms a step
    r = bench.adjoint_ratios({"ratio_backward_over_forward_steps": 1500 / (100 * 5.0)}, 5.0, 3.75)
    assert r == {"adjoint_forward_ratio": 3.0, "adjoint_run_ratio": 4.0}
