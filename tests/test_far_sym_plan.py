"""Host logic of the sums that take every unordered pair once (`csrc/far_plan.h`): over sizes,
kinds, precisions and scratch limits, the workgroups of every phase cover each pair of point
blocks exactly once (the pairs inside a block once as an ordered block), every chunk of a row
has a partial-sum slot of its own below `slots`, the reduction reads exactly the slots that are
written, and the scratch stays within the limit.  The index arithmetic of the kernel and of its
reduction is repeated here from `csrc/k_far_sym.hip`.  Built with g++ from the header alone."""
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
static long bad = 0, planned = 0, refused = 0;
static void check(int N, int kind, int prec, size_t cap) {
  const SymPlan sp = sym_plan(N, kind, prec, cap);
  if (sp.rows < 1) { ++refused; return; }
  ++planned;
  const int nv = kind == 4 ? 6 : kind >= 2 ? 1 : 3;
  const int sg = kind == 4 ? 32 : 64;  // sources per pass of the kernel
  if (sp.tb % sp.csl || sp.tb % sp.css || sp.csl % sg || sp.css % sg || (long)sp.nb * sp.tb < N ||
      (long)(sp.nb - 1) * sp.tb >= N) { ++bad; return; }
  const int pl = sp.tb / sp.csl, ps = sp.tb / sp.css, nb = sp.nb, h = sp.h;
  std::vector<long> seen((size_t)nb * nb, 0);  // sources of block j seen by row i
  for (int row0 = 0; row0 < nb; row0 += sp.rows) {
    const SymPhase ph = sym_phase(sp, std::min(sp.rows, nb - row0));
    if (ph.rows > 65535 * 64 || ph.chunks > 65535) ++bad;
    if (sym_need(sp, ph.rows, nv) > cap) ++bad;
    std::vector<std::vector<char>> slot_used(ph.rows, std::vector<char>(ph.slots, 0));
    std::vector<int> used(ph.rows, 0);
    for (int cy = 0; cy < ph.chunks; ++cy)
      for (int x = 0; x < ph.width; ++x) {
        const int nlong = ph.nl * pl, cs = cy < nlong ? sp.csl : sp.css, per = sp.tb / cs;
        const int jr = cy < nlong ? cy / per : ph.nl + (cy - nlong) / per;
        const int sub = (cy < nlong ? cy : cy - nlong) % per;
        const int r = sym_row(jr, x, nb, h, ph.rows), row = row0 + r;
        if (r < 0) continue;
        if (r >= ph.rows) { ++bad; continue; }
        int j = row0 + jr;
        j -= j >= nb ? nb : 0;
        int o = j - row;
        o += o < 0 ? nb : 0;
        if (o > h) ++bad;
        if (o > 0 && 2 * o == nb && row >= o) continue;
        if (j < 0 || j >= nb || sub >= per) { ++bad; continue; }
        int slot = cy - (r < ph.nl ? r * pl : nlong + (r - ph.nl) * ps);
        slot += slot < 0 ? ph.chunks : 0;
        if (slot < 0 || slot >= ph.slots || slot_used[r][slot]) { ++bad; continue; }
        slot_used[r][slot] = 1;
        ++used[r];
        seen[(size_t)row * nb + j] += cs;
      }
    for (int r = 0; r < ph.rows; ++r) {
      const int jb = row0 + r, no = nb > 1 && 2 * h == nb && jb >= h ? h : h + 1, end = r + no;
      auto first = [&](int j) { return j < ph.nl ? j * pl : ph.nl * pl + (j - ph.nl) * ps; };
      const int n = end <= ph.nj ? first(end) - first(r) : first(ph.nj) - first(r) + first(end - ph.nj);
      if (n != used[r]) ++bad;
      for (int k = 0; k < n && k < ph.slots; ++k) if (!slot_used[r][k]) ++bad;
    }
  }
  for (int i = 0; i < nb; ++i)
    for (int j = i; j < nb; ++j) {
      const long a = seen[(size_t)i * nb + j], b = i == j ? 0 : seen[(size_t)j * nb + i];
      if (a + b != sp.tb) ++bad;
      if (a != 0 && b != 0) ++bad;
    }
}
int main() {
  for (int kind = 0; kind < 5; ++kind)
    for (int prec = 0; prec < 2; ++prec) {
      for (int N = 14000; N <= 60000; N += 509) check(N, kind, prec, sym_cap(N));
      for (int N : {15000, 15360, 15361, 32767, 32768, 49152, 49999, 50000, 50688, 59999, 60000, 119999, 120000, 159901,
                    299999, 300000, 544000})
        for (size_t f : {1, 2, 5, 40}) check(N, kind, prec, sym_cap(N) / f);
      check(1248000, kind, prec, sym_cap(1248000));
      for (int N : {20000, 28000, 32767}) check(N, kind, prec, (size_t)(60.0 * (1 << 17)));
      for (int N : {36000, 40000, 56000, 100000, 160000, 500000, 760000}) check(N, kind, prec, ((size_t(192) << 20) - 120 * (size_t)N) / 8);
    }
  long cap_bad = 0;
  for (long N = 1; N < 5000000; N += N < 200000 ? 1 : 977)
    if (sym_cap(N) > sym_cap(N + 1)) ++cap_bad;
  // below 28,672 points the limit is the no-allocation entry point's too: its 192 MiB hold
  // the packed points and normals, one output and the scratch, in either precision
  for (size_t N = 1; N < 28672; ++N)
    if (N * (64 + 32 + 24) + 3 * 256 + 8 * sym_cap(N) > (size_t(192) << 20)) ++cap_bad;
  std::printf("%ld %ld %ld %ld\n", bad, planned, refused, cap_bad);
  return 0;
}
"""


def test_every_block_pair_is_taken_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = tmp_path / "check"
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    bad, planned, refused, cap_bad = map(int, subprocess.run([str(exe)], check=True, capture_output=True,
                                                             text=True).stdout.split())
    assert bad == 0 and cap_bad == 0
    assert planned > 300 and refused > 0
