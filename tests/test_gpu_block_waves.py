"""The wavefronts reported for blocked launches follow the cells' floes, whatever
batching the per-step kernels are given (needs an MI355X)."""
import pytest

import fixtures

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2303_07819_amd")


@pytest.mark.parametrize("waves", [None, 1, 8])
def test_block_waves_follow_the_largest_cell(waves):
    counts = [0, 3, 64, 65, 128, 129, 200, 300, 513, 700]
    w = fixtures.custom(5, 2, 25e3, counts, seed=3, r_scale=fixtures.radius_scale(700, 25e3 ** 2))
    with sp.Sim.from_workload(w) as s:
        if waves is not None:
            s.set_batching([waves] * sp.NUM_BUCKETS, [0] * sp.NUM_BUCKETS)
        assert s.block_waves().tolist() == [1, 2, 4, 8, 16]
    w = fixtures.custom(2, 1, 25e3, [1, 0], seed=4)
    with sp.Sim.from_workload(w) as s:
        assert s.block_waves().tolist() == [1, 0, 0, 0, 0]
