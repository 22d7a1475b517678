// All-pairs sums between bodies with every unordered pair of points evaluated once.
//
// The kernels of the off-body sums (§2.1, §4) share most of a pair's arithmetic between the
// two directions: d, |d|^2, the reciprocal square root with its correction and the powers
// of |d| serve target a <- source b and target b <- source a alike, only the products with
// the normals and densities differ.  In float64 a traction pair takes 35 operations and one
// v_rsq_f64 for both directions instead of 2 x (24 + 1), the fused traction + Stokeslet pair
// 53 + 1 instead of 2 x (35 + 1), and the sums are bound by VALU issue.
//
// Mapping on gfx950: the points are cut into nb blocks of TB = 256 TPL.  Block row i pairs its
// points with the next h = nb / 2 blocks in cyclic order (for even nb the last of them only
// for i < nb / 2), so every pair of blocks occurs once; the pairs inside block i are
// evaluated in both directions by the ordered path.  A workgroup takes one row and a chunk
// of one block.  Each lane owns TPL points of the row (position, normal, density, sums in
// VGPRs); the chunk's points ("sources") are wave-uniform and arrive by scalar loads, the next
// one while the current one is used.  The contributions to a source are added over the lane's
// TPL points first, then two at a time over lanes 32 apart and (NP = 16) 16 apart by
// v_permlane32_swap and v_permlane16_swap, then in LDS over the remaining lanes and the four
// waves: about 10 operations per source, shared by TPL pairs.  Sums of the row's points go to
// tpart, sums of the sources to spart, both added by k_far_sym_reduce in a fixed order: the
// result does not depend on the order in which workgroups run.  The rows are taken in phases
// of as many rows as the partial-sum buffer holds.
//
// Bound: float64 VALU issue.  Traction, TPL = 6: 38.7 VALU instructions per pair of points (50
// in the ordered kernel for the two directions), VALU busy 0.94 at two waves per SIMD.
// Whole sum with its reductions, MI355X: traction 1,248,000 points 1.21 -> 0.95 s (30 operations
// per ordered pair: 49 TFLOP/s, 0.63 of the 78.6 peak, 0.49 before), 160,000 20.1 -> 15.7 ms,
// 20,000 0.346 -> 0.304 ms; Stokeslet 160,000 18.5 -> 14.9 ms; fused 29.0 -> 25.5 ms; Laplace normal
// derivative and single layer, 73,728 points: 3.07 -> 2.09 and 2.34 -> 1.39 ms; float32
// traction 160,000 9.34 -> 8.41 ms.  Measured slower: full in-wave reduction by DPP with 64
// sources per barrier (the float64 sums 3 % slower, float32 10 %).
//
// Same-body pairs are excluded by body index in the batches that overlap the row's bodies;
// the last, ragged block takes the same masked path.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "far_plan.h"
#include "pair.h"

namespace rbm {

// a and b summed over lanes 32 apart: lanes 0-31 get a's sums, lanes 32-63 b's.
__device__ __forceinline__ float fold32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double fold32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// a and b summed over lanes 16 apart: even rows of 16 lanes get a's sums, odd rows b's.
__device__ __forceinline__ float fold16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// v of the lane 8 apart in the row of 16.
__device__ __forceinline__ float ror8(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));
}
__device__ __forceinline__ double ror8(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x128, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), 0x128, 0xf, 0xf, true));
}

__device__ __forceinline__ double rsq_t(double x) { return __builtin_amdgcn_rsq(x); }
__device__ __forceinline__ float rsq_t(float x) { return __builtin_amdgcn_rsqf(x); }

// Values per point of each kind: traction (0), Stokeslet (1), Laplace normal derivative (2),
// Laplace single layer (3), traction then Stokeslet (4).
__host__ __device__ constexpr int sym_values(int kind) { return kind == 4 ? 6 : kind >= 2 ? 1 : 3; }

// Both directions of one pair: va is the contribution of source b to point a, vb that of point
// a to source b, up to the constants of k_far_sym_reduce (kPost of pair.h, and the sign of
// vb for the kinds odd in d: 0, 2 and the first half of 4).  Same corrections of the hardware
// estimate as in pair.h.
template <typename T, int KIND>
__device__ __forceinline__ void pair_sym(const T* x, const T* n, const T* q, const Src8<T>& s, const Nor4<T>& m,
                                         T* fa, T* fb, T* d) {
  d[0] = x[0] - s.v[0];
  d[1] = x[1] - s.v[1];
  d[2] = x[2] - s.v[2];
  const T r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
  const T y = rsq_t(r2);
  const T y2 = y * y;
  T e = 0;
  if constexpr (sizeof(T) == 8) e = fma(-r2, y2, T(1));
  if constexpr (KIND == 0 || KIND == 4) {
    const T dqb = d[0] * s.v[3] + d[1] * s.v[4] + d[2] * s.v[5];
    const T dqa = d[0] * q[0] + d[1] * q[1] + d[2] * q[2];
    const T dna = d[0] * n[0] + d[1] * n[1] + d[2] * n[2];
    const T dnb = d[0] * m.v[0] + d[1] * m.v[1] + d[2] * m.v[2];
    T base = (y2 * y2) * y;
    if constexpr (sizeof(T) == 8) base *= fma(e, fma(e, T(1.75), T(1)), T(0.4));
    fa[0] = (dna * dqb) * base;
    fb[0] = (dnb * dqa) * base;
    if constexpr (KIND == 4) {
      const T ri = fma(y * e, fma(e, T(0.375), T(0.5)), y);
      const T ri2 = ri * ri;
      fa[1] = ri;
      fa[2] = dqb * ri2;
      fb[2] = dqa * ri2;
    }
  } else if constexpr (KIND == 1) {
    const T dqb = d[0] * s.v[3] + d[1] * s.v[4] + d[2] * s.v[5];
    const T dqa = d[0] * q[0] + d[1] * q[1] + d[2] * q[2];
    T ri = y;
    if constexpr (sizeof(T) == 8) ri = fma(y * e, fma(e, T(0.375), T(0.5)), y);
    const T ri2 = ri * ri;
    fa[1] = ri;
    fa[2] = dqb * ri2;
    fb[2] = dqa * ri2;
  } else if constexpr (KIND == 2) {
    const T dna = d[0] * n[0] + d[1] * n[1] + d[2] * n[2];
    const T dnb = d[0] * m.v[0] + d[1] * m.v[1] + d[2] * m.v[2];
    const T base = (y2 * y) * fma(e, fma(e, T(1.25), T(1)), T(2.0 / 3.0));
    fa[0] = (dna * s.v[3]) * base;
    fb[0] = (dnb * q[0]) * base;
  } else {
    fa[0] = fma(y * e, fma(e, T(0.375), T(0.5)), y);
  }
}

// acc += (or, with FIRST, =) the contribution whose factors f pair_sym formed; qo is the other
// point's density.
template <typename T, int KIND, bool FIRST>
__device__ __forceinline__ void pair_acc(const T* f, const T* d, const T* qo, T ri, T* acc) {
  auto put = [](T& a, T u, T v) { a = FIRST ? u * v : fma(u, v, a); };
  if constexpr (KIND == 0 || KIND == 4)
    for (int c = 0; c < 3; ++c) put(acc[c], f[0], d[c]);
  if constexpr (KIND == 1 || KIND == 4) {
    constexpr int o = KIND == 4 ? 3 : 0;
    for (int c = 0; c < 3; ++c) put(acc[o + c], ri, fma(f[2], d[c], qo[c]));
  }
  if constexpr (KIND == 2) acc[0] = FIRST ? f[0] : acc[0] + f[0];
  if constexpr (KIND == 3) put(acc[0], qo[0], ri);
}

template <typename T, int KIND, int TPL, int WPE, int NP, int FL, int SG>
__global__ __launch_bounds__(256, WPE) void k_far_sym(int N, int M, int nb, int h, int csl, int css, int nl, int slots, int row0,
                                                      int rows, const Src8<T>* __restrict__ src,
                                                      const Nor4<T>* __restrict__ nor,
                                                      double* __restrict__ tpart, double* __restrict__ spart) {
  constexpr int NV = sym_values(KIND), TB = 256 * TPL;
  static_assert((NP == 16 || NP == 32) && SG % FL == 0 && FL % 8 == 0 && 64 % FL == 0, "reduction shape");
  constexpr bool NEED_N = KIND == 0 || KIND == 2 || KIND == 4;
  __shared__ T red[4][NV][FL][NP + 1];  // per wave: NP partial sums of FL sources (odd stride)
  __shared__ T tot[2][4][NV][SG];   // per wave: sums of SG sources
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroup (chunk of block j, place x among the rows that pair with it): consecutive
  // workgroups share the chunk; the first nl blocks from row0 are cut into chunks of csl, the
  // others of css
  const int pl = TB / csl, ps = TB / css, nlong = nl * pl, cy = blockIdx.y;
  const int cs = cy < nlong ? csl : css, per = TB / cs;
  const int jr = cy < nlong ? cy / per : nl + (cy - nlong) / per;
  const int sub = (cy < nlong ? cy : cy - nlong) % per;
  const int r = sym_row(jr, blockIdx.x, nb, h, rows), row = row0 + r;
  if (r < 0) return;
  int j = row0 + jr;
  j -= j >= nb ? nb : 0;
  int o = j - row;
  o += o < 0 ? nb : 0;
  if (o > 0 && 2 * o == nb && row >= o) return;  // the pair of blocks belongs to row - o
  const int b0 = j * TB + sub * cs, b1 = min(N, b0 + cs);
  T x[TPL][3], n[TPL][3], q[TPL][3], acc[TPL][NV];
  int blo_t[TPL];
  const int a0 = row * TB;
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    const int a = min(a0 + t * 256 + tid, N - 1);
    const Src8<T> s = src[a];
    Nor4<T> m{};
    if (NEED_N) m = nor[a];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[t][c] = s.v[c];
      q[t][c] = s.v[3 + c];
      n[t][c] = m.v[c];
    }
#pragma unroll
    for (int c = 0; c < NV; ++c) acc[t][c] = 0;
    blo_t[t] = (a / M) * M;
  }
  if (o == 0) {
    // pairs inside the block: every point of the row against the chunk, one direction
    for (int b = b0; b < b1; ++b) {
      const Src8<T> s = src[b];
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        T p[6] = {0, 0, 0, 0, 0, 0};
        if constexpr (KIND == 4) {
          Pair<T, 0>::add(x[t][0], x[t][1], x[t][2], n[t][0], n[t][1], n[t][2], s, p[0], p[1], p[2]);
          Pair<T, 1>::add(x[t][0], x[t][1], x[t][2], n[t][0], n[t][1], n[t][2], s, p[3], p[4], p[5]);
        } else {
          Pair<T, KIND>::add(x[t][0], x[t][1], x[t][2], n[t][0], n[t][1], n[t][2], s, p[0], p[1], p[2]);
        }
        const bool other = (unsigned)(b - blo_t[t]) >= (unsigned)M;
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[t][c] += other ? p[c] : T(0);
      }
    }
  } else {
    const int last = min(N, a0 + TB) - 1;
    const int blo = (a0 / M) * M, bhi = (last / M + 1) * M;
    const bool full = a0 + TB <= N;
    struct Rec {
      Src8<T> s;
      Nor4<T> m;
    };
    auto load = [&](int b) {
      Rec k;
      k.s = src[b];
      if (NEED_N) k.m = nor[b];
      return k;
    };
    // sums of one source over the lane's points
    auto source = [&](const Rec& k, T* sb) {
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        T fa[3], fb[3], d[3];
        pair_sym<T, KIND>(x[t], n[t], q[t], k.s, k.m, fa, fb, d);
        const T ri = KIND == 3 ? fa[0] : fa[1];
        pair_acc<T, KIND, false>(fa, d, k.s.v + 3, ri, acc[t]);
        if (t == 0)
          pair_acc<T, KIND, true>(fb, d, q[t], ri, sb);
        else
          pair_acc<T, KIND, false>(fb, d, q[t], ri, sb);
      }
    };
    // the same with same-body pairs and the lanes past N left out
    auto source_masked = [&](int b, T* sb) {
#pragma unroll
      for (int c = 0; c < NV; ++c) sb[c] = 0;
      if (b >= b1) return;
      const Rec k = load(b);
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        T fa[3], fb[3], d[3], pa[NV], pb[NV];
        pair_sym<T, KIND>(x[t], n[t], q[t], k.s, k.m, fa, fb, d);
        const T ri = KIND == 3 ? fa[0] : fa[1];
        pair_acc<T, KIND, true>(fa, d, k.s.v + 3, ri, pa);
        pair_acc<T, KIND, true>(fb, d, q[t], ri, pb);
        const bool ok = (unsigned)(b - blo_t[t]) >= (unsigned)M && a0 + t * 256 + tid < N;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          acc[t][c] += ok ? pa[c] : T(0);
          sb[c] += ok ? pb[c] : T(0);
        }
      }
    };
    const size_t width = (size_t)h * TB;
    double* so = spart + (size_t)r * NV * width + (size_t)(o - 1) * TB + sub * cs;
    Rec cur = load(min(b0, N - 1));  // the next source, loaded while the current one is used
    int buf = 0;
    for (int g0 = b0; g0 < b1; g0 += SG, buf ^= 1) {
      for (int b = g0; b < g0 + SG; b += 8) {
        // sums of the batch's sources over the wave: two at a time to 32 lanes each, with NP =
        // 16 four at a time to 16 lanes, then to LDS
        T(*const rw)[FL][NP + 1] = red[wv];
        const int at = (b - g0) % FL;
        auto batch = [&](auto&& one) {
#pragma unroll
          for (int quad = 0; quad < 8; quad += 4) {
            T w[2][NV];
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
              T s0[NV], s1[NV];
              one(b + quad + 2 * pr, s0);
              one(b + quad + 2 * pr + 1, s1);
#pragma unroll
              for (int c = 0; c < NV; ++c) {
                w[pr][c] = fold32(s0[c], s1[c]);
                if (NP == 32) rw[c][at + quad + 2 * pr + (lane >> 5)][lane & 31] = w[pr][c];
              }
            }
            if (NP == 16) {
#pragma unroll
              for (int c = 0; c < NV; ++c)
                rw[c][at + quad + (lane >> 5) + 2 * ((lane >> 4) & 1)][lane & 15] = fold16(w[0][c], w[1][c]);
            }
          }
        };
        if (full && b + 8 <= b1 && (b + 8 <= blo || b >= bhi)) {
          batch([&](int bb, T* sb) {
            const Rec nxt = load(min(bb + 1, N - 1));
            if constexpr (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
            source(cur, sb);
            cur = nxt;
          });
        } else {
          batch(source_masked);
          cur = load(min(b + 8, N - 1));
        }
        if ((b + 8 - g0) % FL == 0) {
          // add the partial sums of FL sources: 64 / FL lanes per source, then across those
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          constexpr int LPS = 64 / FL, PPL = NP / LPS;
          const int k = lane % FL, p0 = lane / FL * PPL;
          T v[NV + (NV & 1)];
          v[NV + (NV & 1) - 1] = 0;
#pragma unroll
          for (int c = 0; c < NV; ++c) {
            T a = rw[c][k][p0];
#pragma unroll
            for (int i = 1; i < PPL; ++i) a += rw[c][k][p0 + i];
            v[c] = a;
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          T* o = &tot[buf][wv][0][0] + (b + 8 - g0) - FL + k;
          if constexpr (LPS == 1) {
#pragma unroll
            for (int c = 0; c < NV; ++c) o[c * SG] = v[c];
          } else if constexpr (LPS == 2) {
#pragma unroll
            for (int c = 0; c < NV; c += 2) {
              const T f = fold32(v[c], v[c + 1]);
              if (c + (lane >> 5) < NV) o[(c + (lane >> 5)) * SG] = f;
            }
          } else if constexpr (LPS == 4) {
#pragma unroll
            for (int c = 0; c < NV; c += 4) {
              const T f = fold32(v[c], c + 1 < NV ? v[c + 1] : T(0));
              const T g = c + 2 < NV ? fold32(v[c + 2], c + 3 < NV ? v[c + 3] : T(0)) : T(0);
              const T e = fold16(f, g);
              const int cc = c + (lane >> 5) + 2 * ((lane >> 4) & 1);
              if (cc < NV) o[cc * SG] = e;
            }
          } else {
            static_assert(LPS == 8, "8 lanes per source");
#pragma unroll
            for (int c = 0; c < NV; c += 4) {
              const T f = fold32(v[c], c + 1 < NV ? v[c + 1] : T(0));
              const T g = c + 2 < NV ? fold32(v[c + 2], c + 3 < NV ? v[c + 3] : T(0)) : T(0);
              T e = fold16(f, g);
              e += ror8(e);
              const int cc = c + (lane >> 5) + 2 * ((lane >> 4) & 1);
              if (cc < NV && !(lane & 8)) o[cc * SG] = e;
            }
          }
        }
      }
      __syncthreads();
      for (int i = tid; i < NV * SG; i += 256) {
        const int c = i / SG, k = i % SG;
        const double v = ((double)tot[buf][0][c][k] + (double)tot[buf][1][c][k]) +
                         ((double)tot[buf][2][c][k] + (double)tot[buf][3][c][k]);
        if (g0 + k < b1) so[c * width + (g0 - b0) + k] = v;
      }
    }
  }
  // the row's chunks in order from its own block on: slots 0, 1, ...
  int slot = cy - (r < nl ? r * pl : nlong + (r - nl) * ps);
  slot += slot < 0 ? (int)gridDim.y : 0;
  double* to = tpart + ((size_t)r * slots + slot) * NV * TB;
#pragma unroll
  for (int t = 0; t < TPL; ++t)
#pragma unroll
    for (int c = 0; c < NV; ++c) to[c * TB + t * 256 + tid] = (double)acc[t][c];
}

// out[c][g] (+)= st (sum of tpart over the chunks of g's row) + ss (sum of spart over the phase's
// rows that have g among their sources), out0 for c < 3 and out1 after.  64 outputs per
// workgroup; the four waves take the terms round-robin and are added in a fixed order.
// Bound by the reads: 0.2 ms for 0.8 GB at 160,000 points (T = 6).
template <int NV>
__global__ __launch_bounds__(256) void k_far_sym_reduce(int N, int tb, int nb, int h, int csl, int css, int nl, int nj,
                                                        int slots, int row0, int rows, int first, double st0,
                                                        double ss0, double st1, double ss1,
                                                        const double* __restrict__ tpart,
                                                        const double* __restrict__ spart,
                                                        double* __restrict__ out0, double* __restrict__ out1) {
  __shared__ double redt[4][64], reds[4][64];
  const int lane = threadIdx.x & 63, qw = threadIdx.x >> 6;
  const int c = blockIdx.y;
  const int g = blockIdx.x * 64 + lane;
  const int jb = (int)(blockIdx.x * 64) / tb, u = g - jb * tb;
  const size_t width = (size_t)h * tb;
  double at = 0.0, as = 0.0;
  const int rt = jb - row0;
  if (rt >= 0 && rt < rows) {
    // chunks of blocks rt .. rt + no - 1 (cyclic over nj): the last block of an even range
    // belongs to the other row of the pair
    const int no = nb > 1 && 2 * h == nb && jb >= h ? h : h + 1;
    const int pl = tb / csl, ps = tb / css, end = rt + no;
    auto first_chunk = [&](int j) { return j < nl ? j * pl : nl * pl + (j - nl) * ps; };
    const int n = end <= nj ? first_chunk(end) - first_chunk(rt)
                            : first_chunk(nj) - first_chunk(rt) + first_chunk(end - nj);
    const double* p = tpart + ((size_t)rt * slots * NV + c) * tb + u;
    for (int k = qw; k < n; k += 4) at += p[(size_t)k * NV * tb];
  }
  for (int r = qw; r < rows; r += 4) {
    const int i = row0 + r;
    int o = jb - i;
    o += o < 0 ? nb : 0;
    if (o < 1 || o > h || (2 * o == nb && i >= o)) continue;
    as += spart[((size_t)r * NV + c) * width + (size_t)(o - 1) * tb + u];
  }
  redt[qw][lane] = at;
  reds[qw][lane] = as;
  __syncthreads();
  if (qw != 0 || g >= N) return;
  const double vt = (redt[0][lane] + redt[1][lane]) + (redt[2][lane] + redt[3][lane]);
  const double vs = (reds[0][lane] + reds[1][lane]) + (reds[2][lane] + reds[3][lane]);
  double* o = (c < 3 ? out0 + (size_t)c * N : out1 + (size_t)(c - 3) * N) + g;
  const double v = (c < 3 ? st0 : st1) * vt + (c < 3 ? ss0 : ss1) * vs;
  *o = first ? v : *o + v;
}

template <typename T, int KIND, int TPL, int WPE, int NP, int FL, int SG>
static hipError_t sym_run(const SymPlan& sp, int N, int M, const void* src, const void* nor, double* part,
                          double* out0, double* out1, hipStream_t st) {
  constexpr int NV = sym_values(KIND);
  if (sp.tb != 256 * TPL || sp.csl % SG || sp.css % SG) return hipErrorInvalidValue;
  constexpr double post0 = Pair<T, KIND == 4 ? 0 : KIND>::kPost;
  constexpr double s0 = post0 * (KIND == 1 || KIND == 3 ? 1.0 / ((KIND == 1 ? 8.0 : 4.0) * RBM_PI)
                                                        : -(KIND == 2 ? 1.0 : 3.0) / (4.0 * RBM_PI));
  constexpr double sgn = KIND == 1 || KIND == 3 ? 1.0 : -1.0;  // kinds 0, 2 and the first half of 4 are odd in d
  constexpr double s1 = 1.0 / (8.0 * RBM_PI);
  for (int row0 = 0; row0 < sp.nb; row0 += sp.rows) {
    const SymPhase ph = sym_phase(sp, std::min(sp.rows, sp.nb - row0));
    double* tpart = part;
    double* spart = part + (size_t)ph.rows * ph.slots * NV * sp.tb;
    k_far_sym<T, KIND, TPL, WPE, NP, FL, SG><<<dim3(ph.width, ph.chunks), 256, 0, st>>>(
        N, M, sp.nb, sp.h, sp.csl, sp.css, ph.nl, ph.slots, row0, ph.rows, static_cast<const Src8<T>*>(src),
        static_cast<const Nor4<T>*>(nor), tpart, spart);
    k_far_sym_reduce<NV><<<dim3((N + 63) / 64, NV), 256, 0, st>>>(
        N, sp.tb, sp.nb, sp.h, sp.csl, sp.css, ph.nl, ph.nj, ph.slots, row0, ph.rows, row0 == 0, s0, sgn * s0, s1, s1,
        tpart, spart, out0, out1);
  }
  return hipGetLastError();
}

// Points per lane (TPL) and the shape of the LDS reduction: TPL as large as the registers of
// two waves per SIMD allow for the sums that are long enough (the exchange of a source's
// sums is shared by TPL pairs), three at the sizes where the blocks would be too few;
// float32 traction keeps five waves per SIMD with three (88 registers).
template <typename T>
hipError_t launch_far_sym(int kind, const SymPlan& sp, int N, int M, const void* src, const void* nor, double* part,
                          double* out0, double* out1, hipStream_t st) {
  if (N < 1 || M < 1 || sp.rows < 1 || (long)sp.nb * sp.tb < N) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 8) {
    if (kind == 0 && sp.tb == 768) return sym_run<T, 0, 3, 3, 16, 16, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 0) return sym_run<T, 0, 6, 2, 16, 16, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 1) return sym_run<T, 1, 3, 3, 16, 16, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 2) return sym_run<T, 2, 4, 2, 16, 16, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 3) return sym_run<T, 3, 4, 2, 16, 16, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 4) return sym_run<T, 4, 3, 2, 16, 16, 32>(sp, N, M, src, nor, part, out0, out1, st);
  } else {
    if (kind == 0) return sym_run<T, 0, 3, 4, 32, 8, 64>(sp, N, M, src, nor, part, out0, out1, st);
    if (kind == 1) return sym_run<T, 1, 3, 4, 32, 8, 64>(sp, N, M, src, nor, part, out0, out1, st);
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_far_sym<double>(int, const SymPlan&, int, int, const void*, const void*, double*, double*,
                                           double*, hipStream_t);
template hipError_t launch_far_sym<float>(int, const SymPlan&, int, int, const void*, const void*, double*, double*,
                                          double*, hipStream_t);

}  // namespace rbm
