"""Threads that read one object out at the same time, each something else, while no
step runs (needs an MI355X).  Bar: every thread gets what a lone thread gets, bit
for bit."""
import threading

import numpy as np
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


def _same(a, b):
    if isinstance(a, dict):
        return all(_same(a[k], b[k]) for k in a)
    if isinstance(a, (tuple, list)):
        return all(_same(x, y) for x, y in zip(a, b))
    return np.array_equal(a, b)


def _together(reads, times=40):
    alone = [f() for f in reads]
    wrong = []

    def work(i):
        for _ in range(times):
            if not _same(reads[i](), alone[i]):
                wrong.append(i)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(reads))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, [(i, wrong.count(i)) for i in sorted(set(wrong))]


@pytest.mark.parametrize("nx,n", [(4, 32), (3, 700)])
def test_simulation(nx, n):
    w = fixtures.custom(nx, nx, 50e3, n, seed=n, r_scale=0.3)
    with sp.Sim.from_workload(w) as s:
        s.step(w.dt, 3)
        s.synchronize()
        _together([s.read_floes, lambda: s.read_moments(sp.MOMENTS_DEM),
                   lambda: s.read_moments(sp.MOMENTS_CONTINUUM), s.stats])


def test_global_dem():
    w = fixtures.custom(1, 1, 400e3, 3000, seed=3, r_scale=0.2)
    with sp.GlobalDEM.from_workload(w) as g:
        g.step(w.dt, 2)
        _together([g.read_floes, g.read_order, lambda: g.coarse_moments(8, 8), lambda: g.coarse_moments(5, 3), g.stats])


def test_network():
    net = sp.MLP()
    net.set_params(np.random.default_rng(1).normal(0, 0.1, sp.MLP_NPARAMS).astype(np.float32))
    _together([net.get_params] * 3)
    net.close()
