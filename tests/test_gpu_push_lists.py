"""The push's collision stage and the MD lists it leaves for the next step.

Every step is compared with the FP64 oracle from the state before it: a
candidate lost or taken twice, or an MD particle left out of a list, shows as a
particle on another path.  Gas pressures from none over few and more candidates
than a push block stages to every particle a candidate (threshold 2^32);
re-binnings of every step, every other and none.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.parity_util import compare_step, oracle_from_state
from tests.test_gpu_parity import TOL, _random_state, _sim

pytestmark = pytest.mark.gpu


def _steps(wl, sim, n):
    tol = TOL[wl["precision"]]
    for k in range(n):
        st = sim.get_state()
        orc = oracle_from_state(wl, st)
        c0 = sim.counters()
        sim.step(1)
        orc.step(1)
        rep = compare_step(wl, sim.get_state(), orc, tol["pos"], tol["vel"], tol["margin"])
        c1 = sim.counters()
        coll = [b - a for a, b in zip(c0["n_collisions"], c1["n_collisions"])]
        md = [b - a for a, b in zip(c0["md_particles"], c1["md_particles"])]
        print(f"  step {k}: collisions {coll} MD {md} flips {rep['flips']}", flush=True)
        assert rep["flips"] <= 3
        yield coll, md


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("p_gas", [0.0, 10.0, 400.0, 2.0e6])
def test_collision_stage(prec, p_gas):
    # 4,096 electrons in the one push block of a 8x4x4-cell box
    wl = W.tiny(nx=8, ny=4, nz=4, ppc=32, p_gas=p_gas, precision=prec)
    sim = _sim(wl)
    sim.set_state(_random_state(wl, 4096, 4000, seed=3))
    T = sim.derived()["T_null"][0]
    assert (T == 0) == (p_gas == 0.0) and (T == 2 ** 32) == (p_gas == 2.0e6)
    for coll, _ in _steps(wl, sim, 2):
        assert (coll[0] == 0) == (p_gas == 0.0)
    sim.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("every", [1, 2, 0])
@pytest.mark.parametrize("box", [(16, 16, 16), (20, 12, 17)])
def test_md_lists_over_steps(prec, every, box):
    nx, ny, nz = box  # five tiles along x leave single tiles per push block
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=3, cutoff=1, Te_eV=12.0, dt=1e-11, precision=prec,
                grains=[[0.4, ny - 0.3, 6.5], [nx / 2 + 0.2, 5.1, 9.5], [nx - 3.1, 2.2, 7.9]])
    sim = _sim(wl, sort_interval=every)
    sim.set_tuning(ion_sort_interval=every)
    n = nx * ny * nz * 3
    sim.set_state(_random_state(wl, n, n // 3, seed=8, near_grain=300))
    met = 0
    for _, md in _steps(wl, sim, 6):
        met += sum(md)
    assert met > 200
    sim.close()
