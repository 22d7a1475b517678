"""Host rule of the fast multipole leaf sums (`csrc/fmm_plan.h`): a power of two of waves by the number of
work items, or down to a quarter of that where the expansions (done by the first wave alone) and the
sources do not share out to more: a tree of a few points per leaf does not fill the chip with waves
that wait.  Built with g++ from the header alone."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1606_07428_amd", "csrc")

CHECK = r"""
#include <cstdio>
#include "fmm_plan.h"
using namespace rbm;
int main() {
  long bad = 0, n = 0;
  for (int P = 2; P <= 16; ++P)
    for (int L = 0; L <= 6; ++L)
      for (long N = 1; N < 3000000; N = N + 1 + N / 7) {
        const int boxes = 1 << (3 * L);
        for (long tasks : {std::min<long>(N, boxes), N / 64 + 1, N / 64 + std::min<long>(N, boxes)}) {
          if (tasks > N) continue;
          const bool far_on = L >= 2;
          const int w = fmm_leaf_waves((int)N, (int)tasks, boxes, P, far_on);
          const double leaves = std::min<double>(boxes, tasks), share = 1 + 27 * N / leaves / (far_on ? fmm_far_cost(P) : 1);
          ++n;
          const int most = tasks >= 4096 ? 4 : tasks >= 2048 ? 8 : kFmmLeafWaves;
          if (w < most / 4 || w > most || (w & (w - 1)) || (w > most / 4 && w > share)) ++bad;
          if (w < most && 2 * w <= share) ++bad;
        }
      }
  if (fmm_leaf_waves(100000, 31919, 32768, 12, true) != 1 || fmm_leaf_waves(71465, 1289, 512, 12, true) != 8 ||
      fmm_leaf_waves(30000, 498, 64, 4, true) != 16 || fmm_leaf_waves(1248000, 21000, 4096, 12, true) != 4 ||
      fmm_leaf_waves(1, 1, 1, 2, false) != 16 || fmm_leaf_waves(5, 0, 1, 2, false) != 16) ++bad;
  std::printf("%ld %ld\n", bad, n);
  return 0;
}
"""


def test_waves_per_item(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    bad, n = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and n > 10000
