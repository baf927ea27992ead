"""The bench line's goals: what the roofline share and its target count agrees."""
import pytest


@pytest.mark.parametrize("flop,direct,met,goal", [
    (50e9, 267e9, False, True),    # few operations, fast: the share is low, the throughput high
    (100e9, 100e9, True, True),
    (20e9, 60e9, False, False),
])
def test_target_and_share_count_the_same_operations(flop, direct, met, goal):
    import bench
    r = bench.goals(flop, direct, 1.0)
    assert r["target_met"] == (r["frac"] >= r["target_frac"]) == met
    assert r["throughput_goal_met"] == goal
    assert r["throughput_goal_met"] == (r["direct_equivalent_tflops"]
                                        >= r["throughput_goal_tflops"])
