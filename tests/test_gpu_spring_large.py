"""The tangential spring in cells near the most floes that a blocked launch's LDS
holds (needs an MI355X): at most 160 KB, the kernel's static arrays included.
Larger cells take one launch per step.  Bars: the route taken; the floe state and
the contact count of both routes bit for bit."""
import numpy as np
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


@pytest.mark.parametrize("schedule,n,blocked", [
    (sp.SCHED_ALLPAIRS, 960, True), (sp.SCHED_ALLPAIRS, 961, False), (sp.SCHED_ALLPAIRS, 992, False),
    (sp.SCHED_ALLPAIRS, 1024, False), (sp.SCHED_BINNED, 928, True), (sp.SCHED_BINNED, 945, False),
    (sp.SCHED_BINNED, 976, False)])
def test_largest_blocked_spring_cell(schedule, n, blocked):
    w = fixtures.custom(2, 1, 25e3, [n, 65], seed=n, r_scale=fixtures.radius_scale(n, 25e3 ** 2))
    rng = np.random.default_rng(n)
    w.u[:] = rng.normal(0, 0.2, w.nfloes)
    w.v[:] = rng.normal(0, 0.2, w.nfloes)
    print(f"{n} floes, schedule {schedule}", flush=True)
    out = []
    for k in (32, 1):
        with sp.Sim.from_workload(w, flags=sp.SP_TANGENTIAL_SPRING, schedule=schedule) as s:
            s.set_step_block(k)
            assert s.step_block()[1] == (blocked and k > 1)
            for steps in (5, 2):
                s.step(w.dt, steps)
            out.append((s.read_floes(), s.stats()["contacts"]))
    for key in out[0][0]:
        assert np.array_equal(out[0][0][key], out[1][0][key]), key
    assert out[0][1] == out[1][1] > 0
