"""Contraction steps of the weight gradient (csrc/mix_members.h, compiled on
the host): never more than a quarter above what the columns need, and the
float32 quotient that finds a column's member is exact over its range."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12144_amd", "csrc")

CHECKER = r"""
#include <cstdio>
#include <initializer_list>
#include "mix_members.h"
using namespace sht::mixm;
int main() {
  for (int B : {1, 2, 3, 4, 7, 16, 33, 64, 256, 1000, 4096})
    for (int mc = 1; mc <= 1024; ++mc) {
      const long long need = (static_cast<long long>(B) * mc + kStep - 1) / kStep;
      if (static_cast<long long>(B) * mc < (1 << 21) && 4LL * steps(B, mc, 1000) > 5 * need) return std::printf("steps %d %d\n", B, mc), 1;
    }
  for (int mc = 1; mc <= 1024; ++mc) {
    volatile float r = 1.f / static_cast<float>(mc);
    for (int b = 0; b * mc < (1 << 21); ++b)
      for (int m : {0, mc / 2, mc - 1})
        if (b * mc + m < (1 << 21) && member_of(b * mc + m, r) != b) return std::printf("member %d %d %d\n", mc, b, m), 1;
  }
  return 0;
}
"""


def test_members(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "members.cpp"
    src.write_text(CHECKER)
    exe = tmp_path / "members"
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
