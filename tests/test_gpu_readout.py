"""Readouts straight into device buffers against the same readouts through the
staging copy (host buffers, and device buffers that no double fits): every
quantity, with grains that share mesh nodes.

What a repeated readout computes anew (the densities and fluxes, summed with
atomics) may differ in its rounding; the rest is the same to the bit.
"""
import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


def _sizes(nn, fn, names):
    per = dict(phi=1, E=3, rho=1, rho_fixed=1, n=2, flux=6)
    return [per[k] * nn if k in per else {"fine_n": 2, "fine_flux": 6, "fine_phi": 1}[k] * fn
            for k in names]


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
@pytest.mark.parametrize("box", [(8, 6, 10), (15, 9, 11)])
def test_readout_targets(prec, box):
    import torch
    from paper_1801_00972_amd import pic as P
    nx, ny, nz = box
    wl = W.tiny(nx=nx, ny=ny, nz=nz, ppc=5, precision=prec, cutoff=1,
                grains=[[3.3, 2.6, 4.5], [3.8, 2.1, 4.9], [nx - 0.4, ny - 0.5, 6.2]])
    sim = _sim(wl)
    cells = (7, 9, 5)
    sim.set_fine_grid((2.0, 1.5, 3.0), 0.5, cells)
    fn, nn = int(np.prod(np.array(cells) + 1)), nx * ny * (nz + 1)
    sim.average(1, 2)
    sim.step(7)
    bits = [("phi", P.PIC_PHI), ("E", P.PIC_E), ("rho", P.PIC_RHO), ("rho_fixed", P.PIC_RHO_FIXED),
            ("n", P.PIC_N), ("flux", P.PIC_FLUX), ("fine_n", P.PIC_FINE_N),
            ("fine_flux", P.PIC_FINE_FLUX), ("fine_phi", P.PIC_FINE_PHI)]
    if prec == "fp64":
        bits = [b for b in bits if b[0] != "rho_fixed"]
    bits.sort(key=lambda b: b[1])
    avg = [b for b in bits if b[0] not in ("E", "rho", "rho_fixed")]
    for chosen, read in ((bits, "fields"), (avg, "average"), (bits[1::2], "fields"), (avg[::2], "average")):
        names, what = [b[0] for b in chosen], sum(b[1] for b in chosen)
        sizes = _sizes(nn, fn, names)

        def get(ptrs, dev):
            if read == "fields":
                P.pic_fields(sim.ctx, 0, what, ptrs, dev)
            else:
                P.pic_average_read(sim.ctx, 0, -1, what, ptrs, dev)

        host = [np.full(s, np.nan) for s in sizes]
        get(host, False)
        aligned = [torch.full((s,), float("nan"), dtype=torch.float64, device="cuda") for s in sizes]
        get(aligned, True)
        raw = [torch.zeros(8 * s + 8, dtype=torch.uint8, device="cuda") for s in sizes]
        odd = [r[4:4 + 8 * s] for r, s in zip(raw, sizes)]
        get(odd, True)
        torch.cuda.synchronize()
        for name, h, a, o in zip(names, host, aligned, odd):
            a, o = a.cpu().numpy(), o.cpu().numpy().tobytes()
            o = np.frombuffer(o, np.float64)
            if read == "average" or name in ("phi", "E", "rho", "rho_fixed", "fine_phi"):
                assert h.tobytes() == a.tobytes() == o.tobytes(), (read, name)
            else:
                big = np.abs(h).max()
                assert np.abs(a - h).max() <= 1e-12 * big and np.abs(o - h).max() <= 1e-12 * big, name
    sim.close()
