"""Blocked launches over cells of every edge count: one wavefront per 64 floes,
a bucket's cells in runs of one number of wavefronts, candidates decided from
the near ones between refreshes (needs an MI355X).

Bars: the floe state, contact counts and DEM statistics of blocked steps equal
those of per-step launches bit for bit (the same per-floe arithmetic); the
continuum within 1e-12 relative (statistics summed in another fixed order).
"""
import numpy as np
import pytest

import fixtures
from metrics import rel_err

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")

EDGES = [0, 1, 2, 63, 64, 65, 127, 128, 129, 192, 193, 256, 257, 320, 511, 512, 513, 576, 640, 1023]


def _ocean(nmodes, L):
    rng = np.random.default_rng(nmodes)
    k = 2 * np.pi / L * rng.integers(-3, 4, (2, nmodes))
    return fixtures.Ocean(u0=0.02, v0=-0.01, kx=k[0], ky=k[1], au=rng.normal(0, 0.1, nmodes),
                          av=rng.normal(0, 0.1, nmodes), phase=rng.uniform(0, 6.28, nmodes))


def _cells(counts, nx, ny, nmodes, drift, seed=7):
    counts = np.asarray(counts, np.int32)
    w = fixtures.custom(nx, ny, 25e3, counts, seed=seed, G=3.5e3, ocean=_ocean(nmodes, nx * 25e3),
                        r_scale=fixtures.radius_scale(max(int(counts.max()), 256), 25e3 ** 2))
    rng = np.random.default_rng(seed)
    w.u[:] = rng.normal(drift, 0.2, w.nfloes)
    w.v[:] = rng.normal(drift, 0.2, w.nfloes)
    w.omega[:] = rng.normal(0, 1e-4, w.nfloes)
    return w


def _both(w, nsteps, schedule, flags=0, continuum=True):
    out = []
    for k in (1, 32):
        with sp.Sim.from_workload(w, flags=flags, schedule=schedule) as s:
            s.set_step_block(k)
            assert s.step_block()[1] == (k > 1)
            s.step(w.dt, nsteps)
            out.append((s.read_floes(), s.read_moments(sp.MOMENTS_DEM), s.read_moments(sp.MOMENTS_CONTINUUM),
                        s.stats()["contacts"]))
    a, b = out
    print(f"{w.nfloes} floes, {nsteps} steps, contacts {a[3]} / {b[3]}", flush=True)
    for key in a[0]:
        assert np.array_equal(a[0][key], b[0][key]), key
    assert np.array_equal(a[1], b[1])
    assert a[3] == b[3]
    if continuum:
        e = rel_err(b[2], a[2], floor=1e-6).max()
        assert e <= 1e-12, e


@pytest.mark.parametrize("schedule", [sp.SCHED_ALLPAIRS, sp.SCHED_BINNED])
@pytest.mark.parametrize("nmodes", [0, 1, 3])
def test_edge_counts(nmodes, schedule):
    _both(_cells(EDGES, 5, 4, nmodes, 0.0), 37, schedule)


@pytest.mark.parametrize("drift", [0.0, 2.0])
def test_runs_of_many_cells_and_fast_floes(drift):
    """More cells of one count than a run needs to stand alone, and floes that
    cross the skin several times within a block (their spin momentum cancels to
    1e-6 of the grid's largest in some cells, below what 1e-12 of the cell's own
    value resolves for any order of summation: no bar on their continuum)."""
    counts = np.repeat([30, 70, 130, 200], 300)
    _both(_cells(counts, 40, 30, 8, drift), 33, sp.SCHED_BINNED, continuum=drift == 0.0)


@pytest.mark.parametrize("schedule", [sp.SCHED_ALLPAIRS, sp.SCHED_BINNED])
def test_edge_counts_with_the_tangential_spring(schedule):
    _both(_cells([0, 1, 64, 65, 128, 129, 256, 257, 320, 511, 512, 200], 4, 3, 2, 0.0), 37, schedule,
          flags=sp.SP_TANGENTIAL_SPRING)
