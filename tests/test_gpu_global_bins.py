"""Global DEM where its search and re-binning leave their common path: many
floes per sub-bin (more candidates than one round reads, more floes than a lane
moves together), 1, 3 and 4 sub-bins a side, walls; coarse grids of ragged runs
and of more cells than the short runs take (needs an MI355X).

Bars: those of test_gpu_global against the oracle (contact counts and floe
counts equal, velocities and statistics within 1e-5 or the storage floor); the
order after every step that of a stable sort by sub-bin.
"""
import numpy as np
import pytest

import fixtures
import oracle
from helpers import frac
from test_gpu_global import _stable_order, compare

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


def crowded(big, side=30, L=120e3, seed=5):
    """side x side small floes on a jittered lattice around one of radius
    big * L at the centre, which sizes the sub-bins."""
    rng = np.random.default_rng(seed)
    g = (np.arange(side) + 0.5) / side
    x, y = (a.ravel() + rng.uniform(-0.02, 0.02, side * side) / side for a in np.meshgrid(g, g))
    away = np.hypot(x - 0.5, y - 0.5) > big + 0.7 / side
    x, y = x[away], y[away]
    n = x.size + 1
    r = rng.uniform(0.45, 0.495, n) * L / side
    x, y = np.append(x, 0.5), np.append(y, 0.5)
    r[-1] = big * L
    u, v = rng.normal(0, 0.3, n), rng.normal(0, 0.3, n)
    w = fixtures.from_arrays(1, 1, L, np.array([n], np.int32), frac(x * L, L), frac(y * L, L), r, rng.uniform(0.5, 2.0, n),
                             u=u, v=v, ocean=fixtures.Ocean(u0=0.05, v0=0.02, kx=np.array([2 * np.pi / L]),
                                                            ky=np.array([-2 * np.pi / L]), au=np.array([0.1]),
                                                            av=np.array([-0.1]), phase=np.array([0.3])))
    w.dt = 30.0
    return w


@pytest.mark.parametrize("big,bins", [(0.2, 1), (0.16, 3), (0.12, 4), (0.045, 11)])
@pytest.mark.parametrize("nxc,nyc", [(7, 5), (1, 9), (300, 257)])
def test_crowded_sub_bins(big, bins, nxc, nyc):
    w = crowded(big)
    gs = compare(w, 5, nxc, nyc)
    assert gs["contacts"] > 0 and gs["bins"] == (bins, bins)


@pytest.mark.parametrize("big", [0.2, 0.16, 0.12])
def test_crowded_sub_bins_between_walls(big):
    compare(crowded(big), 5, 6, 4, flags=sp.SP_WALL_X, oflags=oracle.WALLS_X)


@pytest.mark.parametrize("big", [0.16, 0.12, 0.045])
def test_order_of_crowded_sub_bins(big):
    w = crowded(big)
    with sp.GlobalDEM.from_workload(w) as g:
        prev, _, _ = g.read_order()
        for _ in range(4):
            f = g.read_floes()
            exp, est = _stable_order(prev, f["xi"], f["yi"], g.stats()["bins"])
            g.step(w.dt, 1)
            prev, starts, fb = g.read_order()
            assert np.array_equal(prev, exp) and np.array_equal(starts, est) and fb == 0
