"""Several continuum steps per launch (one workgroup holding the grid, tiles with
halos, single steps on large grids) against one launch per step (needs an
MI355X).  Bars: floe state bit for bit; the continuum within 1e-12 of each
component's largest value (the same update, its statistics summed in another
order)."""
import numpy as np
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 3), (16, 32), (27, 19), (3, 200), (130, 5), (129, 127), (128, 129)])
def test_steps_per_launch(nx, ny, wall):
    rng = np.random.default_rng(nx * 1000 + ny)
    w = fixtures.custom(nx, ny, 25e3, rng.integers(0, 4, nx * ny).astype(np.int32), seed=nx + ny)
    w.u[:] = rng.normal(0, 0.2, w.nfloes)
    w.v[:] = rng.normal(0, 0.2, w.nfloes)
    flags = sp.SP_WALL_X if wall else 0
    with sp.Sim.from_workload(w, flags=flags) as a, sp.Sim.from_workload(w, flags=flags) as b:
        a.set_step_block(1)
        for n in (1, 2, 6, 9, 33):
            a.step(w.dt, n)
            b.step(w.dt, n)
            fa, fb = a.read_floes(), b.read_floes()
            for key in fa:
                assert np.array_equal(fa[key], fb[key]), key
            qa, qb = a.read_moments(sp.MOMENTS_CONTINUUM), b.read_moments(sp.MOMENTS_CONTINUUM)
            scale = np.maximum(np.abs(qa).max(0), 1e-300)
            assert (np.abs(qb - qa).max(0) / scale).max() <= 1e-12, n
        assert a.stats()["max_cfl"] == pytest.approx(b.stats()["max_cfl"], rel=1e-12)
