"""Meshes whose field stage takes two and eight planes a block, with a last run of
planes that is shorter and a last chunk of a plane that is not full, against the
oracle's solve of the same state.
"""
import pytest

from paper_1801_00972_amd import workloads as W
from tests.parity_util import oracle_from_state
from tests.test_gpu_parity import _check_fields, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("nx,ny,nz", [(20, 30, 1400), (36, 50, 2047)])
def test_fields_of_many_planes(prec, nx, ny, nz):
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=1, precision=prec, cutoff=2,
                grains=[[5.3, 6.1, 7.5], [nx - 0.3, 3.2, nz - 3.4]])
    sim = _sim(wl)
    sim.step(1)
    _check_fields(wl, sim, oracle_from_state(wl, sim.get_state()))
    if prec == "fp32r":
        assert sim.counters()["refine_residual"] <= 1e-10
    sim.close()
