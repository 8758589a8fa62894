"""Layout of an interpolation block's local memory (span_lds.h): the nodes'
moments are records of 16 bytes and have to start at a multiple of 16, odd
spans and the 2D mode among them, behind everything else and inside the block.
No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_01305_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "span_lds.h"
using namespace ibmk;
int main() {
  int bad = 0;
  for (int ns = 1; ns <= kPullSpan; ++ns) {
    const int parts = span_parts(ns);
    const size_t at = nodes_at(ns, parts) * sizeof(double);
    const size_t before = (size_t)(2 + 3 + 3 * parts + 4) * ns * sizeof(double);   // G, B, partial sums, R
    if (at % 16 || at < before || at + 16 * 16 * (size_t)ns > interp_span_lds(ns)) {
      std::printf("span %d: moments at byte %zu, %zu bytes before them, block of %zu\n", ns, at, before, interp_span_lds(ns));
      ++bad;
    }
  }
  return bad;
}
"""


def test_moments_of_the_nodes_are_aligned(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "span_lds.cpp", tmp_path / "span_lds"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
