"""Blocked steps of floes that cross the skin several times within a block: the
continuum (needs an MI355X).  Bar: 1e-12 of each component's largest value; some
cells' own spin momentum cancels to far less than the summands' rounding."""
import numpy as np
import pytest

from test_gpu_block_runs import _cells

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


def test_continuum_of_fast_floes():
    w = _cells(np.repeat([30, 70, 130, 200], 300), 40, 30, 8, 2.0)
    q = []
    for k in (1, 32):
        with sp.Sim.from_workload(w, schedule=sp.SCHED_BINNED) as s:
            s.set_step_block(k)
            s.step(w.dt, 33)
            q.append(s.read_moments(sp.MOMENTS_CONTINUUM))
    scale = np.abs(q[0]).max(0)
    assert (scale > 0).all()
    assert (np.abs(q[1] - q[0]).max(0) / scale).max() <= 1e-12
