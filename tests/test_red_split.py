"""How reductions are split over workgroups, on the host: few workgroups for few
elements, a bounded share each for many, within the partials there is room for."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2412_07731_amd", "csrc")

PROG = r"""
#include <cstdio>
#include "red_split.h"
using namespace ahlp;
int main() {
  int last = 0;
  for (long long n = 0; n <= 40000000; n += n < 4000 ? 1 : n < 3000000 ? 997 : 99991) {
    const long long w = red_wgs(n), share = (n + w - 1) / (w > 0 ? w : 1);
    const long long most = n / RED_PARTIALS + 1;
    const bool ok = w >= 1 && w <= RED_PARTIALS && w >= last && (n > 1024 || w == 1) &&
                    share <= (most > 4608 ? most : 4608);
    if (!ok) { printf("%lld elements: %lld workgroups of %lld\n", n, w, share); return 1; }
    last = (int)w;
  }
  return 0;
}
"""


def test_split(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "r.cpp").write_text(PROG)
    subprocess.run([cc, "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "r.cpp"), "-o", str(tmp_path / "r")],
                   check=True)
    r = subprocess.run([str(tmp_path / "r")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
