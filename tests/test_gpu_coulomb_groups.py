"""The Coulomb pass on cells of prescribed counts: none, one, pairs, triplets,
up to the most that a group's lists hold (64 a cell, 512 a group) and one above,
each with every count of the other species; one step against the oracle.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_coulomb import _step_vs_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("counts", [(0, 1, 2, 3, 4, 5, 6, 7), (3, 64, 63, 2, 0, 33, 62, 1),
                                    (64,), (64, 65, 1)])
def test_coulomb_cell_counts(prec, counts):
    from paper_1801_00972_amd.pic import Simulation
    nx, ny, nz = 8, 8, 4
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=66, precision=prec, seed=2)
    wl["coulomb_interval"], wl["coulomb_lnL"] = 1, 2.0e5
    print(f"[case] coulomb cells of {counts} {prec}", flush=True)
    sim = Simulation(wl)
    st = sim.get_state()
    cell = np.arange(nx * ny * nz)
    k = len(counts)
    take = [np.array(counts)[cell % k], np.array(counts)[(cell // k + cell) % k]]
    low = np.stack([cell % nx, cell // nx % ny, cell // (nx * ny)], axis=1).astype(float)
    for s in range(2):
        n = int(take[s].sum())
        p = st[s]["pos"][:n]
        # offsets away from the faces: nobody changes its cell or meets an electrode
        st[s]["pos"] = np.repeat(low, take[s], axis=0) + 0.25 + 0.5 * (p - np.floor(p))
        st[s]["vel"], st[s]["id"] = st[s]["vel"][:n], st[s]["id"][:n]
    sim.set_state(st)
    _step_vs_oracle(sim, wl, prec)
    sim.close()
