"""One launch of the push and the MD motion, or two, on both sides of the size
where the one launch ends (512 resident blocks: 32x32x28 cells, not 32x32x32),
each step against the FP64 oracle from the state before it; and more MD
particles than move four lanes each.
"""
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _random_state, _sim
from tests.test_gpu_push_lists import _steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("box,ppc,near", [((32, 32, 28), 1, 400), ((32, 32, 32), 1, 400),
                                          ((8, 8, 16), 2, 1000), ((16, 16, 16), 16, 60000)])
def test_push_and_md_launches(prec, box, ppc, near):
    nx, ny, nz = box
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=ppc, cutoff=3, precision=prec,
                grains=[[nx / 2, ny / 2, nz / 2], [nx / 2 + 0.7, 0.2, nz / 2 - 2.5]])
    sim = _sim(wl)
    n = nx * ny * nz * ppc
    sim.set_state(_random_state(wl, n, n, seed=5, near_grain=near))
    met = [sum(md) for _, md in _steps(wl, sim, 3)]
    assert min(met) > near / 4
    sim.close()
