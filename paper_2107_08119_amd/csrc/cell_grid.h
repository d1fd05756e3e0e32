// The number of list cells of a periodic box.  Plain C++: no device code.
#pragma once

#include <cmath>

namespace nep {

// Most cells of a grid: what the scan of the cell counts serves (1,024 block
// totals of 1,024 cells each).  Finer grids were scanned only in part, and their
// cell indices passed 2^31 from edges of 7 um on.
constexpr int kMaxCells = 1 << 20;

// Cells of width at least rc along each cell vector, for a box of the given
// perpendicular widths, at most kMaxCells of them (the finest direction is made
// coarser until they are: a cell may be wider than rc, and 2^23 atoms in 2^20
// cells are eight per cell).  False where a direction has fewer than three.
inline bool cell_counts(const double (&width)[3], double rc, int (&nc)[3]) {
  bool cells = true;
  for (int a = 0; a < 3; ++a) {
    const double fit = std::floor(width[a] / (rc * (1.0 + 1e-9)));
    nc[a] = fit < (double)kMaxCells ? (int)fit : kMaxCells;
    if (!(fit >= 3.0)) cells = false;
  }
  if (!cells) {
    nc[0] = nc[1] = nc[2] = 1;
    return false;
  }
  while ((long long)nc[0] * nc[1] * nc[2] > kMaxCells) {
    int most = 0;
    for (int a = 1; a < 3; ++a)
      if (nc[a] > nc[most]) most = a;
    nc[most] -= (nc[most] + 63) / 64;  // the most is above 101
  }
  return true;
}

}  // namespace nep
