"""Host logic of the one-launch ordered sums (`csrc/far_plan.h`): over every size they take, the chunks
cover the points, a thread packs at most one source, and the slots fit the partial-sum buffer
that the sizes of a workspace give (also a larger one's); beyond, they are refused.  Built with
g++ from the header alone."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1606_07428_amd", "csrc")

CHECK = r"""
#include <cstdio>
#include "far_plan.h"
using namespace rbm;
int main() {
  long bad = 0;
  for (int N = 1; N <= kPackingMax; ++N) {
    const int s = far_packing_slots(N);
    if (s < 1) { ++bad; continue; }
    const int chunk = (N + s - 1) / s;
    if (chunk > 256 || (long)chunk * s < N || (size_t)s * N > far_part_cap(N) || s > 65535) ++bad;
  }
  for (int N : {0, -1, kPackingMax + 1, 1 << 20, 2000000000}) bad += far_packing_slots(N) != 0;
  std::printf("%ld\n", bad);
  return bad != 0;
}
"""


def test_packing_plan(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
