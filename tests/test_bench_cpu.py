"""The benchmark's trajectories: the headline's state, without in-plane stiffness, stays finite for some 12 steps."""

import bench


def test_no_trajectory_is_longer_than_its_steps():
    for warmup, steps in ((0, 1), (1, 6), (5, 20), (0, 40), (8, 8), (9, 3)):
        age, oldest, ages = 0, 0, []
        for k in range(warmup + steps):
            if bench.starts_again(k):
                age = 0
            age += 1
            oldest = max(oldest, age)
            ages.append(age)
        assert oldest <= bench.TRAJECTORY_STEPS <= 10
        assert ages[0] == 1


def test_the_default_run_is_one_trajectory():
    assert not any(bench.starts_again(k) for k in range(1 + 6))
