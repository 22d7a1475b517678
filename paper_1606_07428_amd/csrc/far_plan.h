// Source chunks of the all-pairs sums (host side, plain C++): split s < s1 covers c1
// sources from s c1, split s >= s1 covers c2 sources from s1 c1 + (s - s1) c2, each
// clipped to N; a split that starts at or past N is empty and its slot holds zeros.
// Workgroups are dispatched split by split, so the long chunks (85% of the sources, the
// first half of the splits) run first and the grid drains on the short ones.  A grid that
// is resident all at once has nothing to drain and takes equal chunks.
#pragma once
#include <algorithm>
#include <cstddef>

namespace rbm {

struct FarChunks {
  int s1, c1, c2;
};

// Source chunks per all-pairs sum for N points.  The grid has nbx = ceil(N/256) target
// blocks (one target per lane) times `split` source chunks; 256 CUs hold 2048 resident
// 4-wave workgroups, and about six rounds of them balance the waves' finish times
// (measured on MI355X: at 20k points six rounds are 5 % faster in float64 and 12 % in
// float32 than one), so split >= ceil(6 * 2048 / nbx).  Workgroups run split by split and
// every XCD sweeps the sources of the current chunks; at most kChunkSources sources (2 MiB
// of float64 records, half an XCD's 4 MB L2) in the longest chunk keeps that sweep in L2
// instead of streaming the Infinity Cache.  The long chunks of far_chunks hold 1.7 times
// the mean over floor(split / 2) slots, so split >= 1.7 N / kChunkSources + 2 (at 1.25 M
// points 67 chunks instead of 3).  At most 96, and no fewer than kMinSources sources per
// chunk: below 24,000 points the sum is a serial sweep of too few workgroups unless the
// sources are cut finely.  Bounding the split by nbx as well left k_far two workgroups sweeping
// 144 sources each at 288 points (51 us; 4.2 us with 36 chunks) and 400 workgroups at 5,003
// points (89 us; 33 us with 96 chunks); sums of so few points come to it from solves with upsampling
// and from the Laplace kernels, the others take far_packing_slots below.
constexpr int kChunkSources = 32768;
constexpr int kMinSources = 8;
constexpr int kResident = 2048;  // 4-wave workgroups that 256 CUs hold at once

inline int far_l2_split(long N) { return (int)((17 * N + 10L * kChunkSources - 1) / (10L * kChunkSources)) + 2; }

inline int far_split(int N) {
  const int nbx = (N + 255) / 256;
  const int rounds = (6 * kResident + nbx - 1) / nbx;
  const int l2 = N > kChunkSources ? far_l2_split(N) : 1;
  return std::max(1, std::min(std::max(rounds, l2), std::min(96, (N + kMinSources - 1) / kMinSources)));
}

// Bound, non-decreasing in N, of split * points over all sizes up to N: with nbx' target
// blocks the product is at most 96 N', and each of the two lower bounds of the
// split gives at most (6*2048/nbx' + 1) * 256 nbx' or far_l2_split(N') N'.  The partial-sum
// buffer holds that many points' worth of slots.
inline size_t far_part_cap(size_t N) {
  const size_t rounds = (size_t)6 * kResident * 256 + N + 256;
  const size_t l2 = (size_t)far_l2_split((long)N) * N;
  return std::min(96 * N, std::max(rounds, l2));
}

inline FarChunks far_chunks(int N, int nsplit) {
  if (nsplit < 2) return {0, N, N};
  const int s1 = nsplit / 2, s2 = nsplit - s1;
  if ((long)((N + 255) / 256) * nsplit <= kResident) {
    const int c = (N + nsplit - 1) / nsplit;
    return {s1, c, c};
  }
  const long c1 = std::min((17L * N + 20L * s1 - 1) / (20L * s1), (long)N / s1);
  const long rest = N - s1 * c1;
  const long c2 = std::max(1L, (rest + s2 - 1) / s2);
  return {s1, (int)c1, (int)c2};
}

// Ordered sums of few points in one launch (k_far_packing): 64 targets per workgroup, a quarter of its
// chunk of sources per wave; chunks (partial-sum slots) for one round of the 2048 resident workgroups,
// of at least 8 sources a wave and at most 256 (a thread packs one, 16 KiB of LDS); 0: not
// taken.  Whole rbm_far_traction_static, us, with the launches apart (up to 96 chunks for 256
// targets) and with this: float64 300 points 14.7 -> 12.4, 1000 18.4 -> 12.5, 5003 46.0 -> 34.6, 8000
// 80.0 -> 69.5, 10,000 110 -> 102, 12,000 143 -> 148; float32 5003 40 -> 27, 10,000 72 -> 62, 12,000
// 91 -> 84, 16,000 130 -> 136.
constexpr int kPackingMax = 10240;
inline int far_packing_slots(int N) {
  if (N < 1 || N > kPackingMax) return 0;
  const int blocks = (N + 63) / 64, fill = std::min(kResident / blocks, (N + 4 * kMinSources - 1) / (4 * kMinSources));
  return std::max({1, (N + 255) / 256, fill});
}

// ---- the entry point that allocates nothing (rbm_static.cpp) -----------------------------
// Bytes of scratch per GPU, and those that one slot of the ordered sum may take, which set the largest input.
constexpr size_t kStaticBytes = (size_t)192 << 20, kStaticOneSlot = (size_t)64 << 20;

constexpr size_t static_align(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// Scratch of the ordered sum: packed sources, the slots' partial sums, float32 copies of the targets (prec 1).
inline size_t static_bytes(size_t N, int slots, int prec) {
  return static_align(N * (prec == 0 ? 64 : 32)) + static_align((size_t)slots * 3 * N * sizeof(double)) +
         (prec == 0 ? 0 : 2 * static_align(3 * N * sizeof(float)));
}

// The context's split, lowered until it fits.  Below 36,000 points it does; the ordered sum of more is that of
// the sizes whose unordered pairs do not fit, float64 from about 708,500.  (Within 64 MiB instead of all they had one
// slot, a sweep of all sources that leaves L2: 720,000 points 448 -> 412 ms.)
inline int static_split(int N, int prec) {
  int split = far_split(N);
  while (split > 1 && static_bytes((size_t)N, split, prec) > kStaticBytes) --split;
  return split;
}

// ---- sums with every unordered pair of points evaluated once (k_far_sym.hip) -----------
// nb blocks of tb points; block row i pairs with the h next blocks (cyclic), rows of the nb in
// phases of `rows`.  In a phase that starts at row0 the blocks row0 .. row0 + nj - 1 (cyclic) are
// cut into chunks, the first nl of them of csl points and the rest, which run last and let
// the grid drain, of css.  `slots` bounds the chunks of one row.
struct SymPlan {
  int tb, nb, h, csl, css, lead, rows;  // lead: per cent of a phase's blocks that take csl
  bool few;                             // phases of few rounds of the resident workgroups
};
struct SymPhase {
  int rows, nj, nl, chunks, slots, width;  // width: most rows of the phase that pair with one block
};

// Row (from row0) of the phase at place x among those that pair with block jr (from row0), or -1.
// The grid holds these pairs alone: with a place for every row of the phase half of them
// would leave at once, and where the number of rows is a multiple of 32 the rest fall on half
// of the shader engines, which take workgroups in turn (24,000 points, 32 rows: 0.61 ms
// instead of 0.41).  Where phases are a part of the rows, their first and last blocks pair with fewer
// rows and leave places empty: an odd number of places moves those over all engines, unless it or three times
// it is next to a multiple of 32 (48 places, float64, 96,010 points: 8.45 -> 6.36 ms).  In phases of many
// rounds those blocks weigh little, and the numbers as they are keep more of a row's points in the dies' L2 (fused
// sum of 415,584 points 171 ms, with odd numbers 174).
#ifdef __HIPCC__
__host__ __device__
#endif
inline int sym_row(int jr, int x, int nb, int h, int rows) {
  if (h + rows >= nb) {  // the phase's blocks are all nb, cyclic
    if (x > h) return -1;
    const int r = jr - x;
    return r >= 0 ? (r < rows ? r : -1) : (r + nb < rows ? r + nb : -1);
  }
  const int r = (jr < rows ? jr : rows - 1) - x;
  return r >= 0 && jr - r <= h ? r : -1;
}

inline SymPhase sym_phase(const SymPlan& sp, int rows) {
  SymPhase p;
  p.rows = rows;
  p.nj = std::min(sp.nb, sp.h + rows);
  p.nl = (int)((long)p.nj * sp.lead / 100);
  const int pl = sp.tb / sp.csl, ps = sp.tb / sp.css;
  p.chunks = p.nl * pl + (p.nj - p.nl) * ps;
  p.width = p.nj == sp.nb ? sp.h + 1 : std::min(rows, sp.h + 1);
  if (sp.few) {  // see sym_row
    const auto slow = [](int w) { return w % 32 == 1 || w % 32 == 11 || w % 32 == 21 || w % 32 == 31; };
    for (p.width |= 1; slow(p.width); p.width += 2) {}
  }
  p.slots = (1 + sp.h) * pl + (ps - pl) * std::min(1 + sp.h, p.nj - p.nl);
  return p;
}

// Doubles of scratch one phase needs, nv values per point: the chunks' sums of the row's
// points and the sums of the points at the other end.
inline size_t sym_need(const SymPlan& sp, int rows, int nv) {
  return (size_t)rows * nv * sp.tb * (sym_phase(sp, rows).slots + sp.h);
}

// Scratch (doubles) these sums may use at N points, non-decreasing in N: 120 MiB below 28,672
// points, which the scratch of the no-allocation entry point holds too, so that both run the
// same phases there; above, about what a single phase takes, up to 2 GiB.
constexpr int kSymMin = 15000;
inline size_t sym_cap(size_t N) {
  if (N < (size_t)kSymMin) return 0;
  constexpr double kMiB = 131072.0;  // doubles
  if (N < 28672) return (size_t)(120.0 * kMiB);
  const double f = (double)N / 73728.0;
  return (size_t)std::min(std::max(256.0 * kMiB, 300.0 * kMiB * f * f), 2048.0 * kMiB);
}

// Plan for N points within `cap` doubles of scratch; rows = 0 where the ordered sum is to be
// used.  kind: 0 traction, 1 Stokeslet, 2 and 3 Laplace, 4 traction + Stokeslet; prec: 0
// float64, 1 float32.  Where the line lies, measured on MI355X (ms, the ordered sum with its
// combine against this one with its reduction): float64 traction 0.149 / 0.150 at 12,000
// points, 0.250 / 0.216 at 16,000, 0.475 / 0.408 at 24,000, 4.30 / 3.30 at 73,728 and 20.1 / 15.7
// at 160,000; Stokeslet 0.134 / 0.139, 0.225 / 0.203, 0.432 / 0.380, 3.87 / 3.12; Laplace normal
// derivative 3.07 / 2.09 and single layer 2.34 / 1.39 at 73,728; the fused sum 0.483 / 0.496 at
// 20,000, 4.04 / 3.75 at 60,000 and 29.0 / 25.5 at 160,000 (its six sums a side leave two waves
// per SIMD); float32 traction 0.177 / 0.178 at 20,000, 0.606 / 0.572 at 40,000 and 9.34 / 8.41 at
// 160,000 (its ordered kernel issues nearly two VALU operations per four cycles with eight
// waves per SIMD, more than the five waves here reach, which eats half of the gain).
inline SymPlan sym_plan(int N, int kind, int prec, size_t cap) {
  SymPlan sp{};
  const int from = prec ? 36000 : kind == 4 ? 56000 : kSymMin;
  if (N < from || (prec && kind > 1)) return sp;
  sp.tb = kind == 0 && !prec && N >= 50000 ? 1536 : kind == 2 || kind == 3 ? 1024 : 768;
  sp.nb = (int)(((long)N + sp.tb - 1) / sp.tb);
  sp.h = sp.nb / 2;
  const int nv = kind == 4 ? 6 : kind >= 2 ? 1 : 3;
  // chunks (long, short, per cent long) by size: many short ones keep the chip busy at the
  // small end, few long ones spare partial sums at the large one; where the size's own
  // choice does not fit the scratch in one phase the next coarser is taken, then phases
  constexpr int kClasses = 5;
  const int upto[kClasses] = {32000, 50000, 100000, 300000, 2147483647};
  const int c768[kClasses][3] = {{192, 64, 75}, {384, 128, 85}, {768, 128, 80}, {768, 192, 85}, {768, 192, 90}};
  const int c1024[kClasses][3] = {{128, 64, 75}, {256, 128, 80}, {512, 128, 80}, {512, 256, 90}, {1024, 256, 90}};
  const auto most_rows = [&] {  // that fit
    int a = 0, b = sp.nb;
    while (a < b) {
      const int mid = a + (b - a + 1) / 2;
      if (sym_need(sp, mid, nv) <= cap) a = mid; else b = mid - 1;
    }
    return a;
  };
  int cls = 0, lo = 0;
  while (N >= upto[cls]) ++cls;
  for (;; ++cls) {
    const int* c = sp.tb == 1024 ? c1024[cls] : c768[cls];
    sp.csl = cls == 4 && sp.tb == 1536 ? 1536 : c[0];
    sp.css = c[1];
    sp.lead = c[2];
    lo = most_rows();
    if (lo == sp.nb || cls == kClasses - 1 || (cls == 3 && lo > 0)) break;
  }
  const auto finish = [&] {  // equal phases; false: not worth it
    if (lo < 1) return false;
    const int phases = (sp.nb + lo - 1) / lo;
    sp.rows = (sp.nb + phases - 1) / phases;
    // every phase drains the chip once: two rounds of 512 long chunks in each, or the ordered
    // sum; and the grid's second dimension holds 65,535 chunks
    return (phases == 1 || (long)sp.rows * (1 + sp.h) * (sp.tb / sp.csl) >= 2 * 512) &&
           sym_phase(sp, sp.rows).chunks <= 65535;
  };
  // Phases of few rounds of the resident workgroups (5 a CU in float32, 2 in float64), which only the traction
  // sum of the no-allocation entry point has: half the long chunk and more short ones, or each phase ends
  // on a nearly empty round.  Ordered pairs per ns without and with it: float64 112,606 points 1.32 -> 1.50, 190,148 1.41
  // -> 1.54, 400,009 1.42 -> 1.53 (ordered sum 1.25); float32 69,001 2.56 -> 2.77, 93,044 2.58 -> 2.76, 134,224
  // 2.82 -> 2.83, from 150,000 on no more: 250,007 2.90 -> 2.84 (ordered sum 2.69).
  sp.few = lo > 0 && lo < sp.nb && kind == 0 &&
           (long)lo * (1 + sp.h) * (sp.tb / sp.csl) < 8 * 256 * (prec ? 5 : 2);
  if (sp.few && (!prec || N < 150000)) {
    const SymPlan coarse = sp;
    const int rows = lo;
    sp.csl = sp.tb / 2;
    sp.css = prec ? 128 : 192;
    sp.lead = prec ? 80 : 70;
    lo = most_rows();
    if (finish()) return sp;
    sp = coarse;
    lo = rows;
  }
  return finish() ? sp : SymPlan{};
}

}  // namespace rbm
