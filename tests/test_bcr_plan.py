"""Addresses that the group kernel of the cyclic reduction reads at level 0, on the
host: every one lies inside its array, and together they cover it, for pairs with and
without rows at the start, in the middle and at the end."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2412_07731_amd", "csrc")

PROG = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "bcr_plan.h"
// argv: border width, rows of the pairs; the arrays as ahlp_problem_create lays them out
int main(int argc, char** argv) {
  const int n0 = atoi(argv[1]), P = argc - 2, t0 = (n0 + 15) / 16;
  std::vector<int> l;
  for (int j = 0; j < P; ++j) l.push_back(atoi(argv[2 + j]));
  std::vector<long long> off[3];
  long long size[3] = {0, 0, 0}, rows = 0;
  for (int j = 0; j < P; ++j) {
    off[0].push_back(size[0]); size[0] += l[j] * l[j];
    off[1].push_back(size[1]); if (j + 1 < P) size[1] += l[j + 1] * l[j];
    off[2].push_back(rows * n0); rows += l[j];
  }
  size[2] = rows * n0;
  std::vector<char> seen[3];
  for (int k = 0; k < 3; ++k) seen[k].assign(size[k] > 0 ? size[k] : 1, 0);
  for (int j = 0; j < P; ++j)
    for (int kind = 0; kind < 2 + t0; ++kind) {
      if (kind == 1 && j + 1 >= P) continue;
      const int k = kind < 2 ? kind : 2;
      const ahlp::PairTile t = ahlp::pair_tile(kind, l[j], j + 1 < P ? l[j + 1] : 0, n0, off[k][j]);
      for (int a = 0; a < 16; ++a)
        for (int b = 0; b < 16; ++b) {
          const long long at = t.off + ahlp::tile_at(t.sa, t.sb, t.rows, t.cols, a, b);
          if (at < 0 || at >= (long long)seen[k].size()) {
            printf("pair %d kind %d: reads %lld of %zu\n", j, kind, at, seen[k].size());
            return 1;
          }
          if (a < t.rows && b < t.cols) seen[k][at] = 1;
        }
    }
  for (int k = 0; k < 3; ++k)
    for (long long i = 0; i < size[k]; ++i)
      if (!seen[k][i]) { printf("array %d: %lld is not read\n", k, i); return 1; }
  return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROG)
    subprocess.run([cc, "-std=c++17", "-O1", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)
    return str(d / "plan")


@pytest.mark.parametrize("l", [
    [4], [0], [0, 0, 0], [16] * 5, [3, 16, 1, 7],
    [0, 4, 5], [4, 0, 5], [4, 5, 0], [4, 0, 0, 5], [0, 0, 7], [7, 0, 0], [0, 16, 0, 16, 0], [16] * 8 + [0],
], ids=lambda l: "-".join(map(str, l)))
@pytest.mark.parametrize("n0", [0, 1, 16, 17, 64])
def test_reads_stay_inside(plan, n0, l):
    r = subprocess.run([plan, str(n0)] + [str(v) for v in l], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
