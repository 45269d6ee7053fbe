"""Deal of the ring DFT items over the XCDs (csrc/dft_items.h, compiled on the
host): every item of every field group once, the four items that complete a line
of the workspace on one XCD.  Up to eight groups, no XCD has more chunks than
their even share rounded up; over any number, and over many small segments, no
more than an even share of the items plus eight chunks, where some chunk of a
group is empty (where none is, no more than its full chunk a group)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12144_amd", "csrc")

CHECKER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "dft_items.h"
using namespace sht::dfti;
int main() {
  int segs, groups, nk;
  while (std::scanf("%d %d %d", &segs, &groups, &nk) == 3) {
    const int c = chunk(nk), st = step(nk), full = (2 * nk + c - 1) / c;
    std::vector<int> load(kXcds, 0);
    int ok = c % 4 == 0;
    for (int s = 0; s < segs; ++s)
      for (int g = 0; g < groups; ++g) {
        std::vector<int> on(2 * nk, -1);
        for (int x = 0; x < kXcds; ++x)
          for (int e = 0; e < c; ++e) {
            const int i = item(x, s, g, e, c, st);
            if (i >= 2 * nk) continue;
            ok &= on[i] < 0;
            on[i] = x;
            ++load[x];
          }
        for (int i = 0; i < 2 * nk; ++i) ok &= on[i] >= 0 && on[i] == on[i / 4 * 4];
      }
    const int even = (2 * nk * groups * segs + kXcds - 1) / kXcds;
    std::printf("%d %d %d %d %d\n", ok, *std::max_element(load.begin(), load.end()), even, c, full);
  }
}
"""


def test_deal(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "items.cpp"
    src.write_text(CHECKER)
    exe = tmp_path / "items"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    shapes = [(s, g, nk) for s in (1, 3, 64) for g in (1, 2, 7, 8, 9, 36, 125) for nk in (1, 2, 4, 9, 17, 19, 33, 37, 97, 181, 361)]
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % s for s in shapes), check=True, capture_output=True,
                         text=True).stdout.splitlines()
    assert len(out) == len(shapes)
    for shape, line in zip(shapes, out):
        ok, most, even, chunk, full = map(int, line.split())
        assert ok, shape
        groups = shape[0] * shape[1]
        if groups <= 8 and shape[0] == 1:
            assert most <= -(-groups * full // 8) * chunk, (shape, most)
        if full < 8:
            assert most <= even + 8 * chunk, (shape, most, even)
        else:
            assert most <= groups * chunk, (shape, most)
