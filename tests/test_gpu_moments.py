"""The density and flux moments at the edges of its chunks and windows, against the
oracle's moments of the same state: tiles of more slots than a chunk holds,
ragged boxes whose window spans a period, window margins from none to more than
the window holds, and a cell with more particles than a chunk.

Tolerances: a node sums at most m terms in FP64, so the density is within m eps
of the exact sum and the flux within m eps sum|v W|, which is at most about
sqrt(m) of the largest flux times m.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.parity_util import oracle_from_state, rel_inf

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


def _check(sim, wl, most):
    from paper_1801_00972_amd.pic import PIC_FLUX, PIC_N
    st = sim.get_state()
    n, flux = oracle_from_state(wl, st).moments()
    g = sim.fields(0, PIC_N | PIC_FLUX)
    e_n, e_f = rel_inf(g["n"], n), rel_inf(g["flux"], flux)
    print(f"  n {e_n:.2e} flux {e_f:.2e}", flush=True)
    assert e_n <= 4 * most * EPS and e_f <= 4 * most * np.sqrt(most) * EPS


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("nx,ny,nz,ppc,margin", [
    (8, 8, 12, 40, 2), (15, 9, 11, 18, 1), (5, 6, 9, 35, 3), (16, 16, 8, 17, 0)])
def test_moments_chunks_and_windows(prec, nx, ny, nz, ppc, margin):
    from paper_1801_00972_amd.pic import Simulation
    wl = W.tiny(nx, ny, nz, ppc, precision=prec)
    print(f"[case] {wl['name']} {prec} margin {margin}", flush=True)
    sim = Simulation(wl)
    sim.set_tuning(sort_interval=0, ion_sort_interval=0, tile_margin=margin, ion_tile_margin=margin)
    for steps in (0, 5, 20):
        sim.step(steps)
        _check(sim, wl, 8 * 4 * ppc)
    sim.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
def test_moments_one_cell_over_a_chunk(prec):
    from paper_1801_00972_amd.pic import Simulation
    wl = W.tiny(8, 8, 12, 10, precision=prec)
    print(f"[case] {wl['name']} {prec} one cell", flush=True)
    sim = Simulation(wl)
    st = sim.get_state()
    for s in range(2):
        pos = st[s]["pos"]
        st[s]["pos"] = np.array([5.0, 6.0, 7.0]) + (pos - np.floor(pos))
    sim.set_state(st)
    _check(sim, wl, len(st[0]["id"]))
    sim.close()
