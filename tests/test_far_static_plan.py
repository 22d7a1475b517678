"""Host logic of the no-allocation traction sum (`csrc/far_plan.h`): where its sources are summed in order
(below the sizes that take every unordered pair once, and where those do not fit its scratch) it has
the split of the context's sum up to 36,000 points in either precision, so the same result, and
above as many slots as the whole scratch holds.  Built with g++ from the header alone."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1606_07428_amd", "csrc")

CHECK = r"""
#include <cstdio>
#include "far_plan.h"
using namespace rbm;
int main() {
  long bad = 0, lowered = 0, refused = 0;
  for (int prec = 0; prec < 2; ++prec)
    for (int N = 1; static_bytes(N, 1, prec) <= kStaticOneSlot; N += N < 40000 ? 1 : 997) {
      const int s = static_split(N, prec);
      if (s < 1 || s > far_split(N) || static_bytes(N, s, prec) > kStaticBytes) ++bad;
      if (N < 36000 && s != far_split(N)) ++bad;
      if (s < far_split(N)) ++lowered;
      if (s < far_split(N) && static_bytes(N, s + 1, prec) <= kStaticBytes) ++bad;
      const size_t front = (size_t)N * (prec ? 72 : 120) + 768;
      if (N > 100000 && sym_plan(N, 0, prec, std::min(sym_cap(N), (kStaticBytes - front) / 8)).rows < 1) {
        ++refused;
        if (s < 7) ++bad;
      }
    }
  std::printf("%ld %ld %ld\n", bad, lowered, refused);
  return 0;
}
"""


def test_split_of_the_static_sum(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    bad, lowered, refused = map(int, subprocess.run([str(exe)], check=True, capture_output=True,
                                                    text=True).stdout.split())
    assert bad == 0
    assert lowered > 100 and refused > 10
