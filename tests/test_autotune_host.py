"""The autotuner on the stand-in runtime (CPU only): what it reports is the
mean of the launches it was asked for, and every kernel it times runs on
inputs that the kernel before it in a step left -- moments in that schedule's
layout, wall stashes that the step before wrote."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host"))
import standin as S  # noqa: E402


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return S.build(tmp_path_factory.mktemp("standin"))


@pytest.mark.parametrize("reps", [1, 2, 5, 64, 100])
def test_reported_times_are_means_over_reps_launches(lib, reps):
    assert "ok" in S.run(lib, """
import ctypes as C
import standin as S
reps = %d
h = S.Handle([(40, 24, 30, 0)])
n = h.pkg.num_variants()
ms = (C.c_double * (n + 1))()
h.call("autotune", reps, ms)
t = (C.c_double * 100000)()
k = S.standin().standin_elapsed(t, 100000)
assert k >= (n + 1) * reps, k
for v in range(n):
    want = sum(t[v * reps:(v + 1) * reps]) / reps
    assert abs(ms[v] - want) <= 1e-6 * want, (v, ms[v], want)
three = [sum(t[i:i + reps]) / reps for i in range(n * reps, k - reps + 1)]
assert min(abs(ms[n] - x) for x in three) <= 1e-6 * ms[n]
h.close()
print("ok")
""" % reps)


@pytest.mark.parametrize("storage", [0, 1, 3, 4])
def test_candidates_run_on_the_inputs_of_a_step(lib, storage):
    assert "ok" in S.run(lib, """
import standin as S
for walls in (0, 1, 2, 3):
    for model in (3, 0):
        h = S.Handle([(33, 17, 40, walls), (20, 12, 9, walls)], storage=%d, model=model)
        h.call("autotune", 3, None)
        bad = S.faults()
        assert not bad, (walls, model, bad)
        h.call("step", 5)
        if model == 3 or %d in (0, 4):
            h.call("set_schedule", 2, stream=False)
            h.call("step", 5)
        h.close()
        bad = S.faults()
        assert not bad, (walls, model, bad)
print("ok")
""" % (storage, storage))
