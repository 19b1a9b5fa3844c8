// Launches whose grid has a row per item (blockIdx.y).  gfx950 hands a workgroup 16
// bits of its y, so a launch takes at most GRID_ROWS items; more go in several.
// Plain C++, so that the split can be checked on the host.
#pragma once

#include <algorithm>

namespace ahlp {

constexpr int GRID_ROWS = 65535;

// fn(first item, items) for each launch
template <class F>
void grid_rows(int n, F fn) {
  for (int a = 0; a < n; a += std::min(GRID_ROWS, n - a)) fn(a, std::min(GRID_ROWS, n - a));
}

}  // namespace ahlp
