"""Read-outs through the pinned buffer and, beyond its limit, around it: the
same values either way (needs an MI355X)."""
import numpy as np
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


@pytest.mark.parametrize("nx,ny", [(1, 1), (7, 3), (218, 218), (219, 218)])
def test_statistics_on_both_sides_of_the_staging_limit(nx, ny):
    """11 statistics of 47,524 cells fit the 4 MiB buffer, those of 47,742 do
    not; sp_read_moments_noalloc reads around it."""
    w = fixtures.custom(nx, ny, 25e3, np.full(nx * ny, 2, np.int32), seed=4)
    with sp.Sim.from_workload(w) as s:
        s.step(w.dt, 3)
        for which in (sp.MOMENTS_DEM, sp.MOMENTS_CONTINUUM, sp.MOMENTS_DEM):
            assert np.array_equal(s.read_moments(which), s.read_moments_noalloc(which))


@pytest.mark.parametrize("n", [1, 1000, 149795, 149797])
def test_floes_on_both_sides_of_the_staging_limit(n):
    """Seven arrays of 149,795 floes and the error word fit the buffer, those of
    149,797 do not: unmoved floes read back as they were set."""
    rng = np.random.default_rng(n)
    nx = 200
    counts = np.full(nx, n // nx, np.int32)
    counts[: n - counts.sum()] += 1
    w = fixtures.custom(nx, 1, 25e3, np.minimum(counts, 1000), seed=4, r_scale=0.01)
    w.u[:] = rng.normal(0, 0.1, w.nfloes)
    w.theta[:] = rng.uniform(0, 6, w.nfloes)
    with sp.Sim.from_workload(w) as s:
        f = s.read_floes()
    for key in ("xi", "yi", "u", "v", "omega", "theta", "r"):
        assert np.array_equal(f[key], getattr(w, key)), key
