"""Host logic of the sums that take every unordered pair once (`csrc/far_plan.h`): in a phase of
part of the block rows the places of the grid that leave at once are spread over the chip.  Workgroups go in
turn to 8 dies and to 4 shader engines in each, so those whose linear number agrees modulo 32
share an engine; the work (sources) of the fullest is at most 1.1 of the mean, at the sizes of the
no-allocation entry point's scratch.  Built with g++ from the header alone."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1606_07428_amd", "csrc")

CHECK = r"""
#include <cstdio>
#include <vector>
#include "far_plan.h"
using namespace rbm;
int main() {
  double worst = 0;
  int plans = 0;
  for (int prec = 0; prec < 2; ++prec)
    for (int N = 60000; N < 760000; N += N / 97) {
      const size_t front = (size_t)N * (prec ? 72 : 120);
      const SymPlan sp = sym_plan(N, 0, prec, std::min(sym_cap(N), ((size_t(192) << 20) - front) / 8));
      if (sp.rows < 1 || sp.rows >= sp.nb) continue;
      ++plans;
      const SymPhase ph = sym_phase(sp, sp.rows);
      const int pl = sp.tb / sp.csl, ps = sp.tb / sp.css, nlong = ph.nl * pl;
      std::vector<double> work(32, 0.0);
      for (int cy = 0; cy < ph.chunks; ++cy)
        for (int x = 0; x < ph.width; ++x) {
          const int jr = cy < nlong ? cy / pl : ph.nl + (cy - nlong) / ps;
          if (sym_row(jr, x, sp.nb, sp.h, ph.rows) >= 0)
            work[((long)cy * ph.width + x) % 32] += cy < nlong ? sp.csl : sp.css;
        }
      double most = 0, sum = 0;
      for (double w : work) most = std::max(most, w), sum += w;
      worst = std::max(worst, 32 * most / sum);
    }
  std::printf("%.4f %d\n", worst, plans);
  return 0;
}
"""


def test_phases_are_balanced(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    worst, plans = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert float(worst) < 1.1 and int(plans) > 100


CONTEXT = r"""
#include <cstdio>
#include "far_plan.h"
using namespace rbm;
int main() {
  long bad = 0, plans = 0;
  for (int kind = 0; kind < 5; ++kind)
    for (int prec = 0; prec < 2; ++prec)
      for (int N = 14000; N < 6000000; N += N / 400) {
        const SymPlan sp = sym_plan(N, kind, prec, sym_cap(N));
        if (sp.rows < 1) continue;
        ++plans;
        const SymPhase ph = sym_phase(sp, sp.rows);
        if (ph.width != (ph.nj == sp.nb ? sp.h + 1 : std::min(sp.rows, sp.h + 1))) ++bad;
      }
  std::printf("%ld %ld\n", bad, plans);
  return 0;
}
"""


def test_phases_of_a_context_have_no_spare_places(tmp_path):
    """A context's scratch gives phases of many rounds: no more places than rows that pair with a block
    (spare ones move a row's points between the dies' L2 and slowed the fused sum by 1 %)."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "context.cpp"
    src.write_text(CONTEXT)
    exe = tmp_path / "context"
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    bad, plans = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert bad == 0 and plans > 10000
