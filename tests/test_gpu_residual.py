"""The residual record of the FP32R form's solve against NumPy, number for number.

Without grains and with both electrodes at zero the returned potential is the
solve's own psi and the charge density gives its right-hand side to the bit, so
r = b - A psi is formed here with the same operations (the product by six fused,
as longdouble holds it exactly) and only the order of the sums over the nodes
differs.  A block's sums lost, stale or counted twice change ||r|| / ||b|| by
far more.  Solves follow each other with and without a look at the counters in
between: the count of solves above the tolerance rises by one for each of
these, and by none of the others.

Sizes: one plane a block of the field kernel, several (with a remainder of
planes), planes of less than a block and of a ragged number of blocks; the
chunked solve along z and, above 1,024 planes, the serial one.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W

pytestmark = pytest.mark.gpu

EPS0, E = 8.8541878128e-12, 1.602176634e-19
SIZES = [(2, 3, 9), (5, 3, 66), (18, 15, 67), (64, 64, 34), (100, 81, 4), (64, 64, 257), (128, 120, 265),
         (4, 6, 1025), (6, 4, 1026), (2, 3, 2047)]


def _residual(f, nx, ny, nz, dx):
    vol = dx * dx * dx
    scale = -dx * dx / EPS0 * ((E / 4294967296.0) / vol)
    b = scale * f["rho_fixed"].reshape(nz + 1, ny, nx)[1:nz].astype(np.float64)
    p = f["phi"].reshape(nz + 1, ny, nx)
    assert not p[0].any() and not p[nz].any()
    q = p[1:nz]
    s = np.roll(q, -1, 2) + np.roll(q, 1, 2)
    s = s + np.roll(q, -1, 1)
    s = s + np.roll(q, 1, 1)
    s = s + p[2:]
    s = s + p[:-2]
    six = (s.astype(np.longdouble) - np.longdouble(6.0) * q.astype(np.longdouble)).astype(np.float64)
    r = b - six
    return float(np.sqrt((r * r).sum() / (b * b).sum()))


@pytest.mark.parametrize("tol", [1e-10, 1e-30])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_residual_record(size, tol):
    from paper_1801_00972_amd.pic import PIC_PHI, PIC_RHO_FIXED, Simulation
    nx, ny, nz = size
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=1, precision="fp32r", seed=11, V_dc=0.0, V_rf=0.0, refine_tol=tol)
    sim = Simulation(wl)
    seen, above = [], 0

    def look():
        nonlocal above
        f = sim.fields(0, PIC_PHI | PIC_RHO_FIXED)
        seen.append(_residual(f, nx, ny, nz, wl["dx"]))
        above += seen[-1] > tol

    def check():
        c = sim.counters()
        assert c["refine_sweeps"] == 1
        # the summation's own rounding is below 1e-10; a node whose fused product falls
        # on a tie of the 64-bit format moves the norm by less than 1e-6
        assert abs(c["refine_residual"] - seen[-1]) <= 1e-6 * seen[-1]
        assert c["refine_unconverged"] == above

    look()
    check()
    check()  # (a second look adds up nothing again)
    sim.step(1)  # its solve is of the state just read
    above += seen[-1] > tol
    check()
    for _ in range(3):  # solves in a row, each one's sums added up by the next
        look()
        sim.step(1)
        above += seen[-1] > tol
    check()
    look()
    look()
    check()
    sim.step(2)  # (one of the two states was not read)
    look()
    above += 2 * (tol < 1e-20)
    check()
    print(f"  {size}: residuals {seen[0]:.2e} .. {seen[-1]:.2e}, above {above}", flush=True)
    assert len(set(seen)) > 3 or max(seen) == 0.0
    sim.close()
