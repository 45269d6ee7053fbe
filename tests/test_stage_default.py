"""Default staging rule (csrc/stage_default.h, compiled on the host) against
measured shapes where one choice is faster by a tenth or more."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12144_amd", "csrc")

# nlat, lmax, fields: SHT and ISHT together, direct / staged us
DIRECT = [(33, 32, 8), (33, 32, 256), (61, 60, 254), (73, 72, 16), (73, 72, 50), (121, 120, 36), (181, 180, 16),
          (241, 240, 22), (361, 360, 4), (541, 540, 4), (721, 720, 2)]
STAGED = [(33, 32, 1792), (33, 32, 3584), (17, 16, 3584), (61, 60, 728), (73, 72, 707), (121, 120, 364), (181, 180, 364),
          (361, 360, 91), (541, 540, 40), (721, 720, 72)]


def test_measured_shapes(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "stage.cpp"
    src.write_text('#include <cstdio>\n#include "stage_default.h"\nint main() { int n, l, f; while (std::scanf("%d %d %d", '
                   '&n, &l, &f) == 3) std::printf("%d\\n", sht::staging::segment(f, l, (n + 1) / 2)); }\n')
    exe = tmp_path / "stage"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    for shapes, want in ((DIRECT, "0"), (STAGED, "1")):
        out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % s for s in shapes), check=True, capture_output=True,
                             text=True).stdout.split()
        assert out == [want] * len(shapes), list(zip(shapes, out))
