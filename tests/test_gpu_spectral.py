"""The FP64 half-spectrum Poisson solve against a NumPy solve of the same charge.

Sizes at its edges: sides of 2, odd sides (a last row without a partner),
every radix, the largest planes a block takes whole and the smallest it does
not, one row pair or column per block, and each form of the tridiagonal solve.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W

pytestmark = pytest.mark.gpu

EPS0 = 8.8541878128e-12


def _numpy_phi(rho, nx, ny, nz, dx, volt):
    b = np.fft.fft2(-dx * dx / EPS0 * rho.reshape(nz + 1, ny, nx)[1:nz])
    lam = 4 * np.sin(np.pi * np.arange(nx) / nx) ** 2 + 4 * np.sin(np.pi * np.arange(ny) / ny)[:, None] ** 2
    f = np.zeros((nz - 1, ny, nx))
    for k in range(nz - 1):
        f[k] = 1.0 / (-(2.0 + lam) - (f[k - 1] if k else 0.0))
        b[k] = (b[k] - (b[k - 1] if k else 0.0)) * f[k]
    for k in range(nz - 3, -1, -1):
        b[k] -= f[k] * b[k + 1]
    phi = np.zeros((nz + 1, ny, nx))
    phi[1:nz] = np.fft.ifft2(b).real + volt * np.arange(1, nz)[:, None, None] / nz
    phi[nz] = volt
    return phi.reshape(-1)


SIZES = [(2, 2, 2), (3, 5, 7), (5, 3, 66), (15, 9, 67), (25, 27, 12), (30, 36, 129), (64, 64, 34),
         (96, 96, 5), (100, 100, 4), (100, 81, 4), (128, 120, 6), (108, 125, 3), (1024, 2, 3),
         (2, 1024, 3), (1000, 3, 4), (4, 6, 1025), (6, 4, 1026), (2, 3, 2047)]


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_potential_matches_numpy_solve(size, prec):
    from paper_1801_00972_amd.pic import PIC_PHI, PIC_RHO, Simulation
    nx, ny, nz = size
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=1, precision=prec, seed=5)
    if min(nx, ny) >= 3 and nz >= 7:
        wl["grain_pos"] = np.array([[nx / 2 + 0.3, ny - 0.6, nz / 2 + 0.1], [0.2, 0.7, 3.4]])
        wl["cutoff"] = 1
    sim = Simulation(wl)
    if len(wl["grain_pos"]):
        st = sim.get_state()
        st["grain_count"] = np.array([[500, 3], [7, 90]])
        sim.set_state(st)
    # the rounding of a solve: a few eps of the potential, times the condition
    # (nz / pi)^2 of the lowest mode
    tol = 40 * 2.2e-16 * (4 + (nz / np.pi) ** 2)
    for _ in range(2):  # (FP32R: the second solve starts from the first's potential)
        f = sim.fields(0, PIC_PHI | PIC_RHO)
        volt = wl["V_dc"]
        ref = _numpy_phi(f["rho"], nx, ny, nz, wl["dx"], volt)
        err = np.abs(f["phi"] - ref).max() / max(np.abs(ref).max(), 60.0)
        print(f"  {size} {prec}: {err:.1e} of {tol:.1e}", flush=True)
        assert err <= tol
    if prec == "fp32r":
        c = sim.counters()
        assert c["refine_sweeps"] == 1
        assert c["refine_residual"] <= 1e-10 or c["refine_unconverged"] > 0
    sim.close()
