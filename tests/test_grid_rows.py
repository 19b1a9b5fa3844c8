"""The split of launches with a grid row per item, on the host: the parts follow one
another, cover all items and none has more rows than a workgroup's y can number; and
every launch in the library with a row per block goes through it."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2412_07731_amd", "csrc")

PROG = r"""
#include <cstdio>
#include "grid_rows.h"
int main() {
  for (int n : {0, 1, 65534, 65535, 65536, 65537, 131070, 131071, 70000, 2000000}) {
    int at = 0;
    bool ok = true;
    ahlp::grid_rows(n, [&](int first, int count) {
      ok = ok && first == at && count >= 1 && count <= 65535;
      at += count;
    });
    if (!ok || at != n) { printf("%d items\n", n); return 1; }
  }
  return 0;
}
"""


def test_split(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "g.cpp").write_text(PROG)
    subprocess.run([cc, "-std=c++17", "-I", CSRC, str(tmp_path / "g.cpp"), "-o", str(tmp_path / "g")], check=True)
    r = subprocess.run([str(tmp_path / "g")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_launches_with_rows_go_through_it():
    """Grids of two dimensions: a row per block only inside grid_rows (its count), the
    others have a fixed few (a set's reductions, its vectors)."""
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith(".hip"):
            continue
        text = open(os.path.join(CSRC, name)).read()
        for grid in re.findall(r"hipLaunchKernelGGL\([^;]*?dim3\(((?:[^()]|\([^()]*\)|\((?:[^()]|\([^()]*\))*\))*)\)", text):
            depth, parts = 0, [""]
            for ch in grid:
                depth += (ch == "(") - (ch == ")")
                if ch == "," and depth == 0:
                    parts.append("")
                else:
                    parts[-1] += ch
            if len(parts) > 1:
                assert parts[1].strip() in ("count", "k", "s.cnt", "m.nred"), (name, grid)
