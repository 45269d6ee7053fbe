"""Split of a channel mix's zeros (m > l) over workgroups and lanes
(csrc/mix_zeros.h, compiled on the host): every zero is written exactly once,
no column tile writes more than three tiles' worth of columns (or a row per wave), and no wave makes
more than twice the passes that an even share would take (lanes per row are a
power of two) plus the one that rounding up costs.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12144_amd", "csrc")

# batch, channels, mmax, mcount
SHAPES = [(1, 1, 2, 1), (64, 64, 8, 1), (64, 64, 8, 7), (256, 64, 8, 3), (16, 256, 10, 4), (4, 256, 360, 180),
          (4, 256, 360, 359), (1, 677, 360, 1), (1, 33, 65, 32), (3, 5, 22, 21), (2, 130, 129, 64), (5, 7, 100, 33), (16, 1, 360, 90), (4, 32, 360, 45)]

CHECKER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "mix_zeros.h"
using namespace sht::mixz;
int main() {
  int B, C, M, mc;
  while (std::scanf("%d %d %d %d", &B, &C, &M, &mc) == 4) {
    const int tiles = (B * M + 63) / 64, live = (B * mc + 63) / 64, zeros = M - mc;
    for (int r0 = 0; r0 < C; r0 += 128) {
      const int rows = std::min(128, C - r0) * B;
      const Share s = share(tiles, live, rows, zeros);
      std::vector<int> hits(static_cast<size_t>(rows) * zeros, 0);
      long long most_tile = 0, most_passes = 0;
      for (int t = s.first; t < s.first + s.tiles; ++t) {
        long long of_tile = 0;
        for (int w = 0; w < kWaves; ++w) {
          long long passes = 0;
          for (int lane = 0; lane < 64; ++lane) {
            long long n = 0;
            for (int r = first_row(s, t, w, lane); r < rows; r += row_step(s))
              for (int m = first_order(s, lane); m < zeros; m += order_step(s), ++n) ++hits[static_cast<size_t>(r) * zeros + m];
            of_tile += n;
            passes = std::max(passes, n);
          }
          most_passes = std::max(most_passes, passes);
        }
        most_tile = std::max(most_tile, of_tile);
      }
      const long long total = static_cast<long long>(rows) * zeros;
      const int once = std::all_of(hits.begin(), hits.end(), [](int h) { return h == 1; });
      const long long even = (total + 64LL * kWaves * s.tiles - 1) / (64LL * kWaves * s.tiles);
      std::printf("%d %d %lld %lld %lld %d\n", once, s.first + s.tiles <= tiles, most_tile, most_passes, even, rows / B);
    }
  }
}
"""


def test_zero_shares(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "zeros.cpp"
    src.write_text(CHECKER)
    exe = tmp_path / "zeros"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    for shape in SHAPES:
        out = subprocess.run([str(exe)], input=" ".join(map(str, shape)), check=True, capture_output=True, text=True).stdout
        assert out, shape
        for line in out.splitlines():
            once, inside, tile, passes, even, channels = map(int, line.split())
            assert once and inside, shape
            # two tiles' columns and a ragged one, or a row for each wave
            assert tile <= max(3 * 64 * channels, 4 * (shape[2] - shape[3])), shape
            order_passes = -(-(shape[2] - shape[3]) // 64)
            assert passes <= 2 * even + order_passes, (shape, passes, even)
