"""Device buffers that end before the quantity does are refused before anything
is launched, by readouts and averages, whichever of several buffers it is (half as long here); the
context goes on, and the same buffers at their full length are filled.
"""
import ctypes as C

import numpy as np
import pytest

from paper_1801_00972_amd import workloads as W
from tests.test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


class _Raw:
    """One allocation of its own (torch's tensors lie in larger ones), its first bytes
    skipped."""

    def __init__(self, lib, doubles, skip=0):
        self.lib, self.at = lib, C.c_void_p()
        assert lib.hipMalloc(C.byref(self.at), C.c_size_t(8 * doubles + skip)) == 0
        self.skip = skip

    def data_ptr(self):
        return self.at.value + self.skip

    def free(self):
        assert self.lib.hipFree(self.at) == 0


@pytest.mark.parametrize("prec", ["fp64", "fp32r"])
def test_short_device_buffers_are_refused(prec):
    from paper_1801_00972_amd import pic as P
    wl = W.tiny(nx=16, ny=12, nz=40, ppc=2, precision=prec, cutoff=1, grains=[[8.3, 6.1, 20.4]])
    sim = _sim(wl)
    cells = (9, 8, 7)
    sim.set_fine_grid((4.0, 3.0, 16.0), 0.7, cells)
    sim.average(1, 2)
    sim.step(3)
    lib = P.lib()
    nn, fn = sim.n_nodes[0], int(np.prod(np.array(cells) + 1))
    both = [(P.PIC_PHI, nn), (P.PIC_N, 2 * nn), (P.PIC_FLUX, 6 * nn), (P.PIC_FINE_N, 2 * fn),
            (P.PIC_FINE_FLUX, 6 * fn), (P.PIC_FINE_PHI, fn)]
    more = [(P.PIC_PHI, nn), (P.PIC_E, 3 * nn), (P.PIC_RHO, nn)]
    if prec == "fp32r":
        more.append((P.PIC_RHO_FIXED, nn))

    def fields(what, outs):
        P.pic_fields(sim.ctx, 0, what, outs, True)

    def averages(what, outs):
        P.pic_average_read(sim.ctx, 0, -1, what, outs, True)

    for read, quantities in ((fields, more + both[1:]), (averages, both)):
        what = sum(b for b, _ in quantities)
        for short in range(len(quantities)):
            for skip in (0, 8, 4):  # whole, at an offset, and where no double fits
                outs = [_Raw(lib, n // (1 + (k == short)), skip) for k, (_, n) in enumerate(quantities)]
                with pytest.raises(P.PicError) as err:
                    read(what, outs)
                assert err.value.code == P.PIC_EINVAL
                for o in outs:
                    o.free()
        for skip in (0, 8, 4):
            outs = [_Raw(lib, n, skip) for _, n in quantities]
            read(what, outs)
            sim.grain_charges()  # (waits for the stream)
            got = np.zeros(nn)
            assert lib.hipMemcpy(got.ctypes.data_as(C.c_void_p), C.c_void_p(outs[0].data_ptr()),
                                 C.c_size_t(8 * nn), 2) == 0
            assert np.abs(got).max() > 1.0  # the potential
            for o in outs:
                o.free()
    sim.step(1)
    sim.close()
