// Where the group kernel of the cyclic reduction (k_bcr.hip) finds a pair's tiles
// in the assembled Schur complement, level 0.  Plain C++, so that the addresses can
// be checked on the host.
#pragma once

#include "hd.h"

namespace ahlp {

// Tile of one kind of pair j: 0 its diagonal block (in Td), 1 its coupling to the
// next pair (in To), 2 + q tile q of its border rows, transposed (in E).  Element
// (a, b) lies at off + a sa + b sb for a < rows and b < cols.
struct PairTile {
  long long off;
  int sa, sb, rows, cols;
};

// lj, ln: rows of pair j and the next; n0: width of the border; off: where pair j's
// block starts in the kind's array.  A pair may have no rows, and its block then
// starts where the next one does, past the end of the array for the last: a tile
// without elements is taken at the array's start, which always has one value.
AHLP_HD PairTile pair_tile(int kind, int lj, int ln, int n0, long long off) {
  PairTile t{off, 1, lj, lj, lj};
  if (kind == 1) t.sb = t.rows = ln;
  if (kind > 1) t = PairTile{off + 16LL * (kind - 2) * lj, lj, 1, n0 - 16 * (kind - 2), lj};
  if (t.rows <= 0 || t.cols <= 0) t.off = 0;
  return t;
}
// What is read for element (a, b), counted from off: every lane reads, also where the
// tile has no such element.
AHLP_HD int tile_at(int sa, int sb, int rows, int cols, int a, int b) {
  return a < rows && b < cols ? a * sa + b * sb : 0;
}

}  // namespace ahlp
