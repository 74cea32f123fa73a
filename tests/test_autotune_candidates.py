"""The autotuner times no two candidates that launch the same kernels on the same fields,
and times them in calls of the steps that the tuned run makes."""
from paper_2205_02380_amd import autotune, inputs


def _count(grid, reduce, per_call, schedules=("cube", "slab", "plain"), patches=(8,), ghosts=(6,)):
    c = autotune.candidates(grid, 0.02, patches, ghosts, schedules)
    d = autotune.distinct(c, reduce, per_call)
    assert {id(x) for x in d} <= {id(x) for x in c}
    assert sorted(d, key=autotune.accuracy_order) == d
    return len(c), {s: sum(x["schedule"] == s for x in d) for s in schedules}


def test_candidates_that_launch_the_same_are_timed_once():
    g48 = inputs.cubic_grid(48, 16.0, 4, 4.0)            # three tile shapes, two placements
    assert _count(g48, True, 5) == (12, {"cube": 0, "slab": 6, "plain": 6})
    assert _count(g48, False, 1) == (12, {"cube": 0, "slab": 6, "plain": 6})
    assert _count(g48, False, 65) == (12, {"cube": 0, "slab": 6, "plain": 6})
    assert _count(g48, False, 5) == (12, {"cube": 0, "slab": 2, "plain": 6})
    g32 = inputs.cubic_grid(32, 12.0, 4, 4.0)            # one tile shape
    assert _count(g32, True, 5) == (6, {"cube": 2, "slab": 2, "plain": 2})
    for per_call in (1, 5):
        assert _count(g32, False, per_call) == (6, {"cube": 1, "slab": 2, "plain": 2})
    in_place = [c for c in autotune.distinct(autotune.candidates(g32, 0.02, (8,), (6,), ("cube",)), False, 1)]
    assert [c["out_of_place"] for c in in_place] == [False]


def test_results_are_cached_by_the_steps_of_a_call(tmp_path):
    w, path = inputs.workload("C3"), str(tmp_path / "tune.json")
    for n in (0, 1):
        autotune.store(path, w.grid, w.dt, {"reduce_each_step": False, "steps_per_call": n, "best": {"tile": n}})
    assert autotune.lookup(path, w.grid, w.dt)["best"]["tile"] == 0
    assert autotune.lookup(path, w.grid, w.dt, steps_per_call=1)["best"]["tile"] == 1
    assert autotune.lookup(path, w.grid, w.dt, steps_per_call=5) is None
