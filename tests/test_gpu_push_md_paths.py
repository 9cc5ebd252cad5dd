"""Push and MD motion against the FP64 oracle with the path each case names met
for certain: at most 49,152 listed MD particles of a species move four lanes
each, more one lane each, in the one launch of small boxes and in the MD
kernel of its own (32x32x32 cells; which box is which is checked without a GPU).
"""
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _random_state, _sim
from tests.test_gpu_push_lists import _steps

pytestmark = pytest.mark.gpu
QUAD = 49152


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("box,ppc,near", [((16, 16, 16), 16, 60000), ((32, 32, 32), 2, 60000),
                                          ((16, 16, 16), 16, 30000), ((32, 32, 32), 2, 30000)])
def test_lanes_per_md_particle(prec, box, ppc, near):
    nx, ny, nz = box
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=ppc, cutoff=3, precision=prec,
                grains=[[nx / 2, ny / 2, nz / 2], [nx / 2 + 0.7, 0.2, nz / 2 - 2.5]])
    sim = _sim(wl)
    n = nx * ny * nz * ppc
    sim.set_state(_random_state(wl, n, n, seed=6, near_grain=near))
    md = [m for _, m in _steps(wl, sim, 2)]
    for species in range(2):  # (the first step's list holds at least the `near` particles placed)
        assert md[0][species] >= near
        assert (md[0][species] > QUAD) == (near > QUAD)
    sim.close()
