"""The autotuner times no launch twice under two names: the settings it tries
differ in what is launched.
"""
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,replicas", [("fp64", 1), ("fp32r", 1), ("fp32r", 2), ("fp64", 2)])
def test_trials_differ_in_what_is_launched(prec, replicas):
    from paper_1801_00972_amd import pic as P
    wls = [W.tiny(nx=32, ny=32, nz=32, ppc=2, precision=prec, seed=r) for r in range(replicas)]
    sim = _sim(wls[0]) if replicas == 1 else P.Simulation(wls)
    start = sim.tuning()
    trials = P.pic_autotune(sim.ctx, 1)
    keys = [t for t, _ in trials]
    assert len({tuple(sorted(k.items())) for k in keys}) >= 7
    # without effect, so never varied
    assert {k["batch_blocks"] for k in keys} == {start["batch_blocks"]}
    # FP64: three cells' windows are two cells' (1,053 nodes at most)
    assert {k["tile_margin"] for k in keys} == ({1, 2} if prec == "fp64" else {1, 2, 3})
    assert {k["batch_push"] for k in keys} == ({0, 1} if prec == "fp32r" else {0})
    assert {k["use_graphs"] for k in keys} == {0, 1}
    sim.close()
