"""Several continuum steps per launch (one workgroup holding the grid, tiles with
halos, single steps on large grids) against calls of one step, which take one
launch per step (needs an MI355X).  Bars: everything bit for bit: both paths run
the same blocked DEM steps and the same continuum update, whose products are
written out."""
import numpy as np
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 3), (16, 32), (27, 19), (3, 200), (130, 5), (129, 127), (128, 129)])
def test_launches_of_several_steps(nx, ny, wall):
    rng = np.random.default_rng(nx * 1000 + ny)
    w = fixtures.custom(nx, ny, 25e3, rng.integers(0, 4, nx * ny).astype(np.int32), seed=nx + ny)
    w.u[:] = rng.normal(0, 0.2, w.nfloes)
    w.v[:] = rng.normal(0, 0.2, w.nfloes)
    print(f"grid {nx} x {ny}, wall {wall}, {w.nfloes} floes", flush=True)
    out = []
    for together in (False, True):
        with sp.Sim.from_workload(w, flags=sp.SP_WALL_X if wall else 0) as s:
            got = []
            for n in (2, 6, 9, 33):
                for k in [n] if together else [1] * n:
                    s.step(w.dt, k)
                got.append((s.read_floes(), s.read_moments(sp.MOMENTS_CONTINUUM), s.stats()))
            out.append(got)
    for (fa, qa, sa), (fb, qb, sb) in zip(*out):
        for key in fa:
            assert np.array_equal(fa[key], fb[key]), key
        assert np.array_equal(qa, qb)
        assert sa == sb
