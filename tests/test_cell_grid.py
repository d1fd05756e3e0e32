"""The number of list cells of a box (csrc/cell_grid.h), on the host: cells no
narrower than the list cutoff, no more of them than the scan of their counts
serves, and as many as fit where that is no limit."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2107_08119_amd", "csrc")
SOURCE = """#include "cell_grid.h"
extern "C" int counts(const double* w, double rc, int* nc) {
  const double width[3] = {w[0], w[1], w[2]};
  int out[3];
  const bool cells = nep::cell_counts(width, rc, out);
  for (int a = 0; a < 3; ++a) nc[a] = out[a];
  return cells ? 1 : 0;
}
extern "C" int most(void) { return nep::kMaxCells; }
"""


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(SOURCE)
    so = str(d / "grid.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                           str(d / "grid.cpp")])
    lib = ctypes.CDLL(so)

    def call(width, rc):
        nc = (ctypes.c_int * 3)()
        cells = lib.counts((ctypes.c_double * 3)(*width), ctypes.c_double(rc), nc)
        return bool(cells), list(nc)

    assert lib.most() == 1 << 20
    return call


@pytest.mark.parametrize("rc", [0.7, 5.5, 8.5])
@pytest.mark.parametrize("fit", [(3, 3, 3), (7, 4, 12), (101, 102, 101), (102, 102, 101), (102, 103, 102),
                                 (128, 128, 128), (3, 3, 2000000), (1290, 1290, 1290), (2048, 2048, 1024),
                                 (2048, 2048, 2048), (10**7, 10**7, 10**7), (10**11, 4, 4), (3, 10**300, 5)])
def test_cells_of_a_box(grid, rc, fit):
    width = [(f + 0.5) * rc for f in fit]
    cells, nc = grid(width, rc)
    assert cells
    if fit[0] * fit[1] * fit[2] <= 1 << 20:
        assert nc == list(fit)
        return
    total = nc[0] * nc[1] * nc[2]
    assert (1 << 19) < total <= 1 << 20
    for n, w in zip(nc, width):
        assert n >= 3 and w / n >= rc


@pytest.mark.parametrize("width", [(16.0, 16.6, 100.0), (1.0, 1.0, 1.0), (float("nan"), 50.0, 50.0),
                                   (16.6, 10.0**12, 16.0)])
def test_thin_boxes_have_no_cells(grid, width):
    assert grid(width, 5.5) == (False, [1, 1, 1])
