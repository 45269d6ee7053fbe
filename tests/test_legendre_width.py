"""Column width of the Legendre tiles (csrc/legendre_width.h, compiled on the
host): within its limits, never more column chunks than a work item's 16 bits
hold, no second chunk that one tile could have taken where the chip is full, and
small plans spread over enough workgroups."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12144_amd", "csrc")

CHECKER = r"""
#include <cstdio>
#include <initializer_list>
#include "legendre_width.h"
using sht::legw::width;
#define CHECK(x) if (!(x)) return std::printf("%s: groups %d limit %d tiles %lld steps %d others %g -> %d\n", #x, g, limit, t, steps, others, cb), 1
int main() {
  for (int limit : {4, 6, 9})
    for (int steps : {1, 2, 3, 12})
      for (double others : {0.0, 50.0, 1e6})
        for (long long t : {1LL, 2LL, 32LL, 144LL, 240LL, 360LL, 928LL, 1440LL, 4000LL})
          for (int g : {1, 2, 3, 5, 8, 9, 10, 16, 17, 25, 36, 125, 1000, 131072}) {
            const int cb = width(g, limit, t, steps, others), n = (g + cb - 1) / cb;
            CHECK(cb >= 1 && cb <= limit && cb <= g);
            CHECK(n <= 32768);
            if (steps > 2 && t >= 1440 && g <= limit) CHECK(n == 1);
            if (others == 0.0 && t * g <= 128) CHECK(n == (g + 1) / 2);
            if (others == 0.0 && t * g >= 256 && t <= 256) CHECK(t * n >= 64);
          }
  return 0;
}
"""


def test_widths(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "width.cpp"
    src.write_text(CHECKER)
    exe = tmp_path / "width"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
