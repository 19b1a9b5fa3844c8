"""The rule for optional copies of the blocks, on the host: whatever it admits leaves
the device room for what the handle allocates later."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2412_07731_amd", "csrc")

PROG = r"""
#include <cstdio>
#include "copy_room.h"
int main() {
  int yes = 0;
  for (double free = 0; free <= 400; free += 10)
    for (double later = 0; later <= 400; later += 10)
      for (double need = 1; need <= 60; ++need)
        if (ahlp::copy_fits(need, free, later)) {
          ++yes;
          if (free - need < later || need > free / 8) { printf("need %g of %g, later %g\n", need, free, later); return 1; }
        }
  return yes > 1000 ? 0 : 2;
}
"""


def test_room_is_left(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "c.cpp").write_text(PROG)
    subprocess.run([cc, "-std=c++17", "-I", CSRC, str(tmp_path / "c.cpp"), "-o", str(tmp_path / "c")], check=True)
    r = subprocess.run([str(tmp_path / "c")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
