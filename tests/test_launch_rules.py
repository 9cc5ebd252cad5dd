"""CPU checks of the host's launch rules at the edges of their ranges: a C++
program compiled against the library's headers and linked with it prints what
each rule says.  No device call is made."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1801_00972_amd")


def _run(tmp_path, body):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "launch.hpp"\nusing namespace pic;\nint main() {\n' + body + "\n}\n")
    if not os.path.exists(os.path.join(PKG, "libpic.so")):
        from paper_1801_00972_amd import build
        build.build()
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-fsanitize=undefined", "-I/opt/rocm/include",
                    "-I", os.path.join(PKG, "csrc"), str(src), "-o", str(exe),
                    os.path.join(PKG, "libpic.so"), "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib"], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, check=True)
    assert "runtime error" not in res.stderr, res.stderr
    return [int(x) for x in res.stdout.split()]


@pytest.mark.parametrize("slots,first", [((4 << 20, 4 << 20), 0), ((4 << 20, (4 << 20) + 4), 1),
                                         ((1 << 30, 1 << 30), 1), ((2 ** 31 - 4, 2 ** 31 - 4), 1), ((0, 1024), 0)])
def test_long_pushes_go_first(tmp_path, slots, first):
    assert _run(tmp_path, "WorkLists L[2]{}; L[0].slots = %d; L[1].slots = %d;\n"
                          'std::printf("%%d\\n", (int)push_goes_first(L));' % slots) == [first]


@pytest.mark.parametrize("box,f64,same", [
    ((64, 64, 64), 1, [0, 0, 1]),   # tile pairs in FP64: three cells shrink to two everywhere
    ((36, 32, 64), 1, [0, 0, 0]),   # single tiles: three cells fit at the electrodes
    ((8, 8, 64), 1, [0, 0, 0]),     # a pair's window spans the period: three cells fit
    ((64, 64, 64), 0, [0, 0, 0]),   # (FP32R pairs: 15 x 11 x 8 nodes at the electrodes)
    ((2, 2, 2), 0, [1, 1, 1]),      # the whole box in any window
])
def test_margins_of_the_same_windows(tmp_path, box, f64, same):
    nx, ny, nz = box
    body = "WorkLists L{}; L.ntx = %d; L.nty = %d; L.ntz = %d; L.ngrid = tile_grid(%d, %d, %d, 0);\n" % (
        (nx + 3) // 4, (ny + 3) // 4, (nz + 3) // 4, nx, ny, nz)
    body += 'for (int m = 0; m < 3; ++m) std::printf("%%d\\n", (int)same_windows(L, %d, %d, %d, m, m + 1, %d));' % (
        nx, ny, nz, f64)
    assert _run(tmp_path, body) == same


@pytest.mark.parametrize("box,ppc,one", [((32, 32, 28), 1, 1), ((32, 32, 32), 1, 0), ((8, 8, 16), 2, 1),
                                         ((16, 16, 16), 16, 1), ((32, 32, 32), 2, 0)])
def test_boxes_of_one_launch(tmp_path, box, ppc, one):
    """The boxes that the GPU tests of push and MD motion take lie on the side of the
    one-launch limit that they name (two grains apart, cubes of 7 cells)."""
    nx, ny, nz = box
    cells = 2 * 343 if ny > 8 else 7 * 8 * 7 * 2  # (8 cells: the cubes of 7 overlap; a bound is enough)
    body = "WorkLists L{}; L.ntx = %d; L.nty = %d; L.ntz = %d; L.ngrid = tile_grid(%d, %d, %d, 0);\n" % (
        (nx + 3) // 4, (ny + 3) // 4, (nz + 3) // 4, nx, ny, nz)
    body += "L.slots = (%d + 4 * L.ngrid + 1023) / 1024 * 1024;\n" % (nx * ny * nz * ppc)
    body += "MdTables md{}; md.n_grains = 2; md.n_cells = %d;\n" % cells
    body += "SpeciesStep S{}; S.nx = %d; S.ny = %d; S.nz = %d;\n" % box
    body += 'std::printf("%d\\n", (int)push_md_fits(md, S, L));'
    assert _run(tmp_path, body) == [one]
