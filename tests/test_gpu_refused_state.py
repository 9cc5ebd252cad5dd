"""A state that pic_set_state refuses leaves the context as it was: also one whose
FP32 offsets would round a particle onto the rf electrode, in either species.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _random_state, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("species", [0, 1])
def test_state_rounding_onto_the_electrode_changes_nothing(species):
    from paper_1801_00972_amd import pic as P
    nz = 14
    wl = W.tiny(nx=12, ny=8, nz=nz, ppc=2, precision="fp32r", cutoff=1, grains=[[5.2, 4.4, 6.3]])
    n = 12 * 8 * nz * 2
    sims = [_sim(wl) for _ in range(2)]
    for sim in sims:
        sim.set_state(_random_state(wl, n, n, seed=4, near_grain=40))
        sim.step(3)
    bad = _random_state(wl, n, n, seed=9)
    bad[species]["pos"][n // 2, 2] = nz - 1e-12
    before = sims[0].get_state()
    with pytest.raises(P.PicError) as err:
        sims[0].set_state(bad)
    assert err.value.code == P.PIC_ENUMERIC
    bad[species]["pos"][n // 2, 2] = nz - 2.0 ** -24  # (the largest offset below one)
    after = sims[0].get_state()
    for sim in sims:
        sim.step(9)
    a, b = sims[0].get_state(), sims[1].get_state()
    for s in range(2):
        ia, ib = np.argsort(a[s]["id"]), np.argsort(b[s]["id"])
        for key in ("pos", "vel", "id"):
            assert np.array_equal(before[s][key], after[s][key])
            assert np.array_equal(a[s][key][ia], b[s][key][ib])
    assert np.array_equal(a["grain_count"], b["grain_count"]) and a["step"] == b["step"]
    sims[0].set_state(bad)
    got = sims[0].get_state()[species]
    assert got["pos"][np.flatnonzero(got["id"] == bad[species]["id"][n // 2])[0], 2] == nz - 2.0 ** -24
    for sim in sims:
        sim.close()
