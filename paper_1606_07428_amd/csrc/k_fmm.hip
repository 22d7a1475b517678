// Fast multipole evaluation of the off-body traction sum, an O(N) equivalent of the FMM
// the paper uses for the far field (§3.1).
//
// Stokes through four harmonic potentials: phi_j = sum q_j / |x - y| (j = 1..3) and
// psi = sum ((y - c).q) / |x - y| with c the centre of the box that carries the
// expansion.  At a target x in a leaf with centre c, s = x - c:
//   traction = (1/4pi) [ (div phi) N + (H(psi) - s_j H(phi_j)) N ]      (H: Hessian),
// which is the traction [-pI + grad u + grad u^T] N of the Stokeslet field (§2.1).
//
// Complex solid harmonics with factorial normalisation (no Condon-Shortley phase):
//   R_n^m = r^n P_n^m e^{i m phi} / (n+m)!,  I_n^m = (n-m)! P_n^m e^{i m phi} / r^{n+1},
//   X_n^{-m} = (-1)^m conj(X_n^m); expansions store m >= 0 only, coefficient n(n+1)/2 + m,
//   the four densities of a coefficient adjacent.
// Multipole about c: M_n^m = sum q conj(R_n^m(y - c)); local about c: phi = sum L conj(R(x - c)).
//   M2M (child c1 -> parent c2): M'_n^m = sum_{k,l} M_k^l conj(R_{n-k}^{m-l}(c1 - c2))
//   M2L (a = c_t - c_s):          L_k^l  = (-1)^k sum_{n,m} M_n^m I_{n+k}^{m+l}(a)
//   L2L (parent c -> child c'):   L'_j^i = sum_{k,l} L_k^l conj(R_{k-j}^{l-i}(c' - c))
//   d/dz of a local expansion shifts L_{k+1}^l, (d/dx + i d/dy) shifts L_{k+1}^{l+1}.
// Moving the psi expansion from centre c to c' adds (c - c') . (phi_1, phi_2, phi_3)
// expansions: before the translation in M2M and L2L, after it (by linearity) in M2L.
//
// Tree: uniform octree over the bounding cube of the points (side D, corner lo), leaf
// level L with leaf width >= the largest body diameter, so the nodes of one body lie in
// the same or adjacent leaves: every same-body pair falls in the direct near field,
// where it is skipped; none goes through an expansion.  Near field: the 27 adjacent
// leaves.  Interaction lists at levels 2..L: boxes not adjacent whose parents are.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "fmm.h"
#include "fmm_plan.h"
#include "kernels.h"
#include "pair.h"

namespace rbm {

constexpr int kFmmPMax = kFmmMaxOrder;
constexpr int kFmmKc = (kFmmPMax + 1) * (kFmmPMax + 2) / 2;          // coefficients, m >= 0
constexpr int kFmmLeafMax = kFmmLeafCap;                              // points per leaf
constexpr int kFmmVecs = 343;                                         // displacements in [-3, 3]^3

template <typename T>
__device__ __forceinline__ void cfma(Cx<T>& acc, Cx<T> a, Cx<T> b) {
  acc.re = fma(a.re, b.re, fma(-a.im, b.im, acc.re));
  acc.im = fma(a.re, b.im, fma(a.im, b.re, acc.im));
}

// Entry (n, m) of a half table, any sign of m: X_n^{-m} = (-1)^m conj(X_n^m).
template <typename T>
__device__ __forceinline__ Cx<T> cget(const Cx<T>* a, int n, int m) {
  if (m >= 0) return a[tri(n, m)];
  const Cx<T> v = a[tri(n, -m)];
  return (m & 1) ? Cx<T>{-v.re, v.im} : Cx<T>{v.re, -v.im};
}

// R_n^m(x, y, z) for 0 <= m <= n <= P into out[tri(n, m)] (conjugated if conj):
//   R_m^m = R_{m-1}^{m-1} (x + iy) / (2m),  R_{m+1}^m = z R_m^m,
//   R_n^m = ((2n - 1) z R_{n-1}^m - r^2 R_{n-2}^m) / ((n - m)(n + m)).
template <typename T, typename S>
__device__ void regular_table(int P, S x, S y, S z, Cx<T>* out, bool conj) {
  const S r2 = x * x + y * y + z * z;
  S dre = 1, dim = 0;
  const S sg = conj ? S(-1) : S(1);
  for (int m = 0; m <= P; ++m) {
    if (m > 0) {
      const S inv = S(1) / S(2 * m);
      const S nre = (dre * x - dim * y) * inv, nim = (dre * y + dim * x) * inv;
      dre = nre;
      dim = nim;
    }
    out[tri(m, m)] = Cx<T>{(T)dre, (T)(sg * dim)};
    if (m + 1 > P) continue;
    S are = dre, aim = dim;            // R_{n-2}
    S bre = z * dre, bim = z * dim;    // R_{n-1}
    out[tri(m + 1, m)] = Cx<T>{(T)bre, (T)(sg * bim)};
    for (int n = m + 2; n <= P; ++n) {
      const S c1 = S(2 * n - 1), inv = S(1) / S((n - m) * (n + m));
      const S vre = (c1 * z * bre - r2 * are) * inv, vim = (c1 * z * bim - r2 * aim) * inv;
      are = bre; aim = bim;
      bre = vre; bim = vim;
      out[tri(n, m)] = Cx<T>{(T)vre, (T)(sg * vim)};
    }
  }
}

// I_n^m(x, y, z) for 0 <= m <= n <= Q into out[n^2 + n + m] and, by I_n^{-m} =
// (-1)^m conj(I_n^m), out[n^2 + n - m] (all m, (Q + 1)^2 entries):
//   I_0^0 = 1/r,  I_m^m = I_{m-1}^{m-1} (2m - 1)(x + iy) / r^2,  I_{m+1}^m = (2m + 1) z I_m^m / r^2,
//   I_n^m = ((2n - 1) z I_{n-1}^m - (n + m - 1)(n - m - 1) I_{n-2}^m) / r^2.
template <typename T>
__device__ void irregular_table(int Q, double x, double y, double z, Cx<T>* out) {
  const double r2 = x * x + y * y + z * z, ir2 = 1.0 / r2;
  double dre = 1.0 / sqrt(r2), dim = 0.0;
  auto put = [&](int n, int m, double re, double im) {
    out[n * n + n + m] = Cx<T>{(T)re, (T)im};
    if (m > 0) out[n * n + n - m] = (m & 1) ? Cx<T>{(T)-re, (T)im} : Cx<T>{(T)re, (T)-im};
  };
  for (int m = 0; m <= Q; ++m) {
    if (m > 0) {
      const double c = (2 * m - 1) * ir2;
      const double nre = (dre * x - dim * y) * c, nim = (dre * y + dim * x) * c;
      dre = nre;
      dim = nim;
    }
    put(m, m, dre, dim);
    if (m + 1 > Q) continue;
    double are = dre, aim = dim;
    double bre = (2 * m + 1) * z * ir2 * dre, bim = (2 * m + 1) * z * ir2 * dim;
    put(m + 1, m, bre, bim);
    for (int n = m + 2; n <= Q; ++n) {
      const double c1 = (2.0 * n - 1.0) * z, c2 = (double)(n + m - 1) * (double)(n - m - 1);
      const double vre = (c1 * bre - c2 * are) * ir2, vim = (c1 * bim - c2 * aim) * ir2;
      are = bre; aim = bim;
      bre = vre; bim = vim;
      put(n, m, vre, vim);
    }
  }
}

// ---------------------------------------------------------------------------------
// Tree construction (float64 coordinates)

// Componentwise min and max of this workgroup's share of X ([3][N], first = true), or of earlier
// results X ([N][6]), into out[6 blockIdx.x ..].  Bound: HBM; one workgroup for all points read at 55
// GB/s (1,248,000 points: 0.55 ms, two launches over the chip 0.014).
template <bool FIRST>
__global__ void __launch_bounds__(256) k_fmm_bounds(int N, const double* __restrict__ X, double* out) {
  __shared__ double red[6][256];
  double v[6] = {1e300, 1e300, 1e300, -1e300, -1e300, -1e300};
  for (int i = blockIdx.x * 256 + threadIdx.x; i < N; i += gridDim.x * 256)
    for (int d = 0; d < 3; ++d) {
      v[d] = fmin(v[d], FIRST ? X[(size_t)d * N + i] : X[6 * i + d]);
      v[3 + d] = fmax(v[3 + d], FIRST ? X[(size_t)d * N + i] : X[6 * i + 3 + d]);
    }
  for (int d = 0; d < 6; ++d) red[d][threadIdx.x] = v[d];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int d = 0; d < 6; ++d)
        red[d][threadIdx.x] = d < 3 ? fmin(red[d][threadIdx.x], red[d][threadIdx.x + s])
                                    : fmax(red[d][threadIdx.x], red[d][threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x < 6) out[6 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// counter[key] += 1 for the active lanes of a wave; every lane's old value (the order among lanes of one
// key is that of the lanes).  Consecutive points are a body's, which lies in a few leaves: one
// addition for all lanes of a key, for the first four keys; atomics of single lanes on one address
// run one after the other (1,248,000 points: counting 0.27 -> 0.010 ms, scattering 0.36 -> 0.010).
__device__ __forceinline__ int wave_count(int key, bool active, int* counter) {
  unsigned long long todo = __ballot(active);
  const int lane = threadIdx.x & 63;
  int pos = 0;
  for (int r = 0; r < 4 && todo; ++r) {
    const int leader = __ffsll(todo) - 1, k = __builtin_amdgcn_readlane(key, leader);
    const unsigned long long same = __ballot(key == k) & todo;
    int base = 0;
    if (lane == leader) base = atomicAdd(counter + k, __popcll(same));
    base = __builtin_amdgcn_readlane(base, leader);
    if (same >> lane & 1) pos = base + __popcll(same & ((1ull << lane) - 1));
    todo &= ~same;
  }
  if (todo >> lane & 1) pos = atomicAdd(counter + key, 1);
  return pos;
}

__device__ __forceinline__ int leaf_coord(double x, double lo, double w, int nb) {
  const int i = (int)floor((x - lo) / w);
  return i < 0 ? 0 : (i >= nb ? nb - 1 : i);
}

__global__ void k_fmm_count(int N, const double* __restrict__ X, double lox, double loy, double loz,
                            double w, int nb, int* __restrict__ leaf, int* __restrict__ cnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < N;
  int id = 0;
  if (live) {
    const int a = leaf_coord(X[i], lox, w, nb);
    const int b = leaf_coord(X[(size_t)N + i], loy, w, nb);
    const int c = leaf_coord(X[2 * (size_t)N + i], loz, w, nb);
    id = (c * nb + b) * nb + a;
    leaf[i] = id;
  }
  wave_count(id, live, cnt);
}

// Exclusive scan of cnt[0, nbox) into start[0, nbox]; largest count to *maxcnt.
__global__ void __launch_bounds__(1024) k_fmm_scan(int nbox, const int* __restrict__ cnt,
                                                   int* __restrict__ start, int* __restrict__ maxcnt) {
  __shared__ int part[1024], pmax[1024];
  const int t = threadIdx.x, nt = blockDim.x;
  const int chunk = (nbox + nt - 1) / nt;
  const int b0 = min(nbox, t * chunk), b1 = min(nbox, b0 + chunk);
  int s = 0, mx = 0;
  for (int b = b0; b < b1; ++b) {
    s += cnt[b];
    mx = max(mx, cnt[b]);
  }
  part[t] = s;
  pmax[t] = mx;
  __syncthreads();
  if (t == 0) {
    int run = 0, m = 0;
    for (int i = 0; i < nt; ++i) {
      const int v = part[i];
      part[i] = run;
      run += v;
      m = max(m, pmax[i]);
    }
    start[nbox] = run;
    *maxcnt = m;
  }
  __syncthreads();
  int run = part[t];
  for (int b = b0; b < b1; ++b) {
    start[b] = run;
    run += cnt[b];
  }
}

__global__ void k_fmm_scatter(int N, const int* __restrict__ leaf, const int* __restrict__ start,
                              int* __restrict__ fill, int* __restrict__ perm) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < N;
  const int b = live ? leaf[i] : 0;
  const int at = wave_count(b, live, fill);
  if (live) perm[start[b] + at] = i;
}

// Order every leaf's segment of perm by point index (the atomic scatter leaves it in
// arbitrary order): rank of each entry = number of smaller entries in the segment.
__global__ void __launch_bounds__(256) k_fmm_sort(const int* __restrict__ start, int* __restrict__ perm) {
  __shared__ int v[kFmmLeafMax];
  const int b = blockIdx.x;
  const int s0 = start[b], n = start[b + 1] - s0;
  if (n <= 1 || n > kFmmLeafMax) return;
  for (int i = threadIdx.x; i < n; i += blockDim.x) v[i] = perm[s0 + i];
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int x = v[i];
    int r = 0;
    for (int k = 0; k < n; ++k) r += v[k] < x;
    perm[s0 + r] = x;
  }
}

// Sorted geometry: Xs[p] = (x, y, z, body), Ns[p] = (nx, ny, nz, 0) of point perm[p].
__global__ void k_fmm_gather(int N, int M, const int* __restrict__ perm, const double* __restrict__ X,
                             const double* __restrict__ Nn, double4* __restrict__ Xs,
                             double4* __restrict__ Ns) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const int i = perm[p];
  Xs[p] = make_double4(X[i], X[(size_t)N + i], X[2 * (size_t)N + i], (double)(i / M));
  Ns[p] = make_double4(Nn[i], Nn[(size_t)N + i], Nn[2 * (size_t)N + i], 0.0);
}

// Points per box one level up: cp[parent] = sum of its eight children's counts.
__global__ void k_fmm_level_count(int np, const int* __restrict__ cc, int* __restrict__ cp) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= np * np * np) return;
  const int i = b % np, j = (b / np) % np, k = b / (np * np);
  const int nc = 2 * np;
  int s = 0;
  for (int o = 0; o < 8; ++o) {
    const int ci = 2 * i + (o & 1), cj = 2 * j + ((o >> 1) & 1), ck = 2 * k + (o >> 2);
    s += cc[(ck * nc + cj) * nc + ci];
  }
  cp[b] = s;
}

// Translation tables of levels 2..L (child width w = D / 2^lev):
//   tabR[lev][o] = conj(R(t_o)), t_o = ((o_x - 1/2) w, (o_y - 1/2) w, (o_z - 1/2) w) (child
//   centre minus parent centre, used by M2M into level lev - 1 and by L2L into level lev);
//   tabI[lev][v] = I(v w) for v in [-3, 3]^3 with max |v_i| >= 2 (M2L), degree 2P, all m
//   ((2P + 1)^2 entries, n^2 + n + m).
template <typename T>
__global__ void k_fmm_tables(int P, int L, double D, int nv, Cx<T>* __restrict__ tabR, Cx<T>* __restrict__ tabI) {
  const int lev = 2 + blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (lev > L || e >= 8 + nv) return;
  const int Kc = tri(P + 1, 0), F2 = (2 * P + 1) * (2 * P + 1);
  const double w = ldexp(D, -lev);
  if (e < 8) {
    const double tx = ((e & 1) - 0.5) * w, ty = (((e >> 1) & 1) - 0.5) * w, tz = ((e >> 2) - 0.5) * w;
    regular_table<T, double>(P, tx, ty, tz, tabR + ((size_t)(lev - 2) * 8 + e) * Kc, true);
  } else {
    const int v = e - 8;
    const int vx = v % 7 - 3, vy = (v / 7) % 7 - 3, vz = v / 49 - 3;
    if (abs(vx) <= 1 && abs(vy) <= 1 && abs(vz) <= 1) return;
    irregular_table<T>(2 * P, vx * w, vy * w, vz * w, tabI + ((size_t)(lev - 2) * kFmmVecs + v) * F2);
  }
}

// ---------------------------------------------------------------------------------
// Expansions: [box][Kc][density 0..3] complex (the four densities of one coefficient are
// adjacent, so a wave-uniform reader takes them in one scalar load), density 3 = psi.

// Entry (n, m), any sign of m, of density d of an interleaved expansion.
template <typename T>
__device__ __forceinline__ Cx<T> cget4(const Cx<T>* a, int n, int m, int d) {
  if (m >= 0) return a[tri(n, m) * 4 + d];
  const Cx<T> v = a[tri(n, -m) * 4 + d];
  return (m & 1) ? Cx<T>{-v.re, v.im} : Cx<T>{v.re, -v.im};
}

__device__ __forceinline__ void tri_inv(int c, int& n, int& m) {
  n = (int)((sqrtf(8.0f * c + 1.0f) - 1.0f) * 0.5f);
  while (tri(n + 1, 0) <= c) ++n;
  while (tri(n, 0) > c) --n;
  m = c - tri(n, 0);
}

// Column m (n = m..P) of conj(R_n^m(x, y, z)) into out[tri(n, m)]: the recurrences of
// regular_table for one m, in the same order, so the entries are the same.
template <typename T>
__device__ void regular_column(int P, int m, T x, T y, T z, Cx<T>* out) {
  const T r2 = x * x + y * y + z * z;
  T dre = 1, dim = 0;
  for (int k = 1; k <= m; ++k) {
    const T inv = T(1) / T(2 * k);
    const T nre = (dre * x - dim * y) * inv, nim = (dre * y + dim * x) * inv;
    dre = nre;
    dim = nim;
  }
  out[tri(m, m)] = Cx<T>{dre, -dim};
  if (m + 1 > P) return;
  T are = dre, aim = dim;
  T bre = z * dre, bim = z * dim;
  out[tri(m + 1, m)] = Cx<T>{bre, -bim};
  for (int n = m + 2; n <= P; ++n) {
    const T c1 = T(2 * n - 1), inv = T(1) / T((n - m) * (n + m));
    const T vre = (c1 * z * bre - r2 * are) * inv, vim = (c1 * z * bim - r2 * aim) * inv;
    are = bre; aim = bim;
    bre = vre; bim = vim;
    out[tri(n, m)] = Cx<T>{vre, -vim};
  }
}

// points per P2M chunk (the chunk's tables fill 39 KB of LDS in either precision)
template <typename T> struct P2mChunk { static constexpr int v = sizeof(T) == 8 ? 16 : 32; };

// Leaf multipoles: M_d[c] = sum_p charge_d(p) conj(R_c(y_p - centre)), charges
// (q_x, q_y, q_z, (y - centre).q), sources in leaf order.  One workgroup per leaf, 4 Kc
// threads (one output each, density fastest).  The regular tables of a chunk of points
// are built one (point, m) column per thread, then every output sums over the chunk in
// point order.
template <typename T>
__global__ void __launch_bounds__(1024) k_fmm_p2m(int P, int nb, double lox, double loy, double loz, double w,
                                                  const int* __restrict__ start, const int* __restrict__ perm,
                                                  const double4* __restrict__ Xs, const Src8<T>* __restrict__ src,
                                                  Cx<T>* __restrict__ Mout) {
  constexpr int CH = P2mChunk<T>::v;
  __shared__ Cx<T> Rt[CH][kFmmKc];
  __shared__ T ch[CH][4];
  __shared__ T sp[CH][3];
  const int b = blockIdx.x;
  const int Kc = tri(P + 1, 0);
  const int i = b % nb, j = (b / nb) % nb, k = b / (nb * nb);
  const double cx = lox + (i + 0.5) * w, cy = loy + (j + 0.5) * w, cz = loz + (k + 0.5) * w;
  const int s0 = start[b], n = start[b + 1] - s0;
  const int o = threadIdx.x;
  const int d = o & 3, c = min(o >> 2, Kc - 1);
  const bool live = o < 4 * Kc;
  Cx<T> acc{0, 0};
  for (int base = 0; base < n; base += CH) {
    const int cnt = min(CH, n - base);
    if (o < cnt) {
      const int p = s0 + base + o;
      const double4 x = Xs[p];
      const Src8<T> s = src[p];
      const T sx = (T)(x.x - cx), sy = (T)(x.y - cy), sz = (T)(x.z - cz);
      ch[o][0] = s.v[3];
      ch[o][1] = s.v[4];
      ch[o][2] = s.v[5];
      ch[o][3] = sx * s.v[3] + sy * s.v[4] + sz * s.v[5];
      sp[o][0] = sx;
      sp[o][1] = sy;
      sp[o][2] = sz;
    }
    __syncthreads();
    for (int t = o; t < cnt * (P + 1); t += blockDim.x) {
      const int q = t / (P + 1), m = t - q * (P + 1);
      regular_column<T>(P, m, sp[q][0], sp[q][1], sp[q][2], Rt[q]);
    }
    __syncthreads();
    if (live)
      for (int q = 0; q < cnt; ++q) {
        acc.re = fma(ch[q][d], Rt[q][c].re, acc.re);
        acc.im = fma(ch[q][d], Rt[q][c].im, acc.im);
      }
    __syncthreads();
  }
  if (live) Mout[((size_t)b * Kc + c) * 4 + d] = acc;
}

// Multipoles of level lev - 1 from their eight children at level lev (side nc).
template <typename T>
__global__ void __launch_bounds__(1024) k_fmm_m2m(int P, int nc, double wc, const int* __restrict__ cntc,
                                                  const Cx<T>* __restrict__ tabR, const Cx<T>* __restrict__ Mc,
                                                  Cx<T>* __restrict__ Mp) {
  __shared__ Cx<T> Mch[4][kFmmKc];
  __shared__ Cx<T> Rt[kFmmKc];
  const int np = nc / 2, b = blockIdx.x;
  const int Kc = tri(P + 1, 0);
  const int i = b % np, j = (b / np) % np, k = b / (np * np);
  const int o = threadIdx.x, d = o & 3, c = min(o >> 2, Kc - 1);
  const bool live = o < 4 * Kc;
  int n = 0, m = 0;
  tri_inv(c, n, m);
  Cx<T> acc{0, 0};
  for (int e = 0; e < 8; ++e) {
    const int ci = 2 * i + (e & 1), cj = 2 * j + ((e >> 1) & 1), ck = 2 * k + (e >> 2);
    const int cb = (ck * nc + cj) * nc + ci;
    if (cntc[cb] == 0) continue;
    const T tx = (T)(((e & 1) - 0.5) * wc), ty = (T)((((e >> 1) & 1) - 0.5) * wc), tz = (T)(((e >> 2) - 0.5) * wc);
    const Cx<T>* src = Mc + (size_t)cb * 4 * Kc;
    for (int q = threadIdx.x; q < Kc; q += blockDim.x) {
      const Cx<T> a = src[4 * q], bb = src[4 * q + 1], cc = src[4 * q + 2], dd = src[4 * q + 3];
      Mch[0][q] = a;
      Mch[1][q] = bb;
      Mch[2][q] = cc;
      // psi moves from the child centre to the parent's: + (c1 - c2) . phi
      Mch[3][q] = Cx<T>{dd.re + tx * a.re + ty * bb.re + tz * cc.re, dd.im + tx * a.im + ty * bb.im + tz * cc.im};
      Rt[q] = tabR[(size_t)e * Kc + q];
    }
    __syncthreads();
    if (live)
      for (int kk = 0; kk <= n; ++kk)
        for (int l = max(-kk, m - (n - kk)); l <= min(kk, m + (n - kk)); ++l)
          cfma(acc, cget(Mch[d], kk, l), cget(Rt, n - kk, m - l));
    __syncthreads();
  }
  if (live) Mp[((size_t)b * Kc + c) * 4 + d] = acc;
}

// Locals from the interaction lists (M2L), every level 2..L in one launch: workgroup g
// takes box g - first[lev] of level lev (side nl = 2^lev, width w = D / 2^lev), boxes
// without points are skipped.  One thread per local coefficient (k, l), l >= 0, for all four
// densities, so every table entry a thread reads serves four products.  The source
// multipoles are the same for the whole workgroup: they are read in their stored half
// (m >= 0) with wave-uniform (scalar) loads, the four densities of a coefficient in one, and
// the m < 0 half enters through X_n^{-m} = (-1)^m conj(X_n^m), which pairs the terms of +m
// and -m:  M I_a + (-1)^m conj(M) I_b = M.re (I_a.re + s I_b.re) + ..., four real FMAs per
// density and stored coefficient instead of eight.  The irregular table of the
// displacement (all m) is staged in LDS.  The psi shift from the source centre to the
// target's (- a . phi) is applied after the translation, by linearity:
// T(psi - a.phi) = T(psi) - a . T(phi).  The parents' locals are added afterwards (L2L).
// Float64, and float32 above order kFmmRotOrder; otherwise k_fmm_m2l_rot takes its place.
template <typename T>
__global__ void __launch_bounds__(256) k_fmm_m2l(int P, int L, double D, FmmLevels lv,
                                                 const Cx<T>* __restrict__ tabI, const Cx<T>* __restrict__ Mexp,
                                                 Cx<T>* __restrict__ Lexp) {
  constexpr int kFull2 = (2 * kFmmPMax + 1) * (2 * kFmmPMax + 1);
  __shared__ Cx<T> It[kFull2];
  int lev = 2;
  while (lev < L && (int)blockIdx.x >= lv.first[lev + 1]) ++lev;
  const int b = (int)blockIdx.x - lv.first[lev];
  const int* cnt = lv.cnt[lev];
  if (cnt[b] == 0) return;
  const int nl = 1 << lev;
  const double w = ldexp(D, -lev);
  const int Kc = tri(P + 1, 0), F2 = (2 * P + 1) * (2 * P + 1);
  const Cx<T>* Mlev = Mexp + lv.off[lev] * 4 * Kc;
  const Cx<T>* tabl = tabI + (size_t)(lev - 2) * kFmmVecs * F2;
  const int i = b % nl, j = (b / nl) % nl, k = b / (nl * nl);
  const int c = threadIdx.x;
  const bool act = c < Kc;
  int kk = 0, ll = 0;
  if (act) tri_inv(c, kk, ll);
  Cx<T> acc[4];
  for (int d = 0; d < 4; ++d) acc[d] = Cx<T>{0, 0};
  const T sk_sign = (kk & 1) ? T(-1) : T(1);
  const int pi = i / 2, pj = j / 2, pk = k / 2;
  for (int sk = max(0, 2 * pk - 2); sk <= min(nl - 1, 2 * pk + 3); ++sk)
    for (int sj = max(0, 2 * pj - 2); sj <= min(nl - 1, 2 * pj + 3); ++sj)
      for (int si = max(0, 2 * pi - 2); si <= min(nl - 1, 2 * pi + 3); ++si) {
        const int vx = i - si, vy = j - sj, vz = k - sk;
        if (abs(vx) <= 1 && abs(vy) <= 1 && abs(vz) <= 1) continue;
        const int sb = (sk * nl + sj) * nl + si;
        if (cnt[sb] == 0) continue;
        const Cx<T>* tv = tabl + (size_t)(((vz + 3) * 7 + (vy + 3)) * 7 + (vx + 3)) * F2;
        __syncthreads();  // the previous source's table has been read
        for (int q = threadIdx.x; q < F2; q += blockDim.x) It[q] = tv[q];
        __syncthreads();
        if (act) {
          Cx<T> pt[4];
          for (int d = 0; d < 4; ++d) pt[d] = Cx<T>{0, 0};
          // M I_a + sg conj(M) I_b for the stored coefficient M (four densities at v)
          auto pair = [&](const Cx<T>* v, int ia, int ib, T sg) {
            const Cx<T> ip = It[ia], im = It[ib];
            const T s1 = fma(sg, im.re, ip.re), s2 = fma(sg, im.im, -ip.im);
            const T s3 = fma(sg, im.im, ip.im), s4 = fma(-sg, im.re, ip.re);
            for (int d = 0; d < 4; ++d) {
              const Cx<T> a = v[d];
              pt[d].re = fma(a.re, s1, fma(a.im, s2, pt[d].re));
              pt[d].im = fma(a.re, s3, fma(a.im, s4, pt[d].im));
            }
          };
          // the source's coefficients in stored order: (n, 0), (n, 1), ..., (n, n), (n + 1, 0), ...
          const Cx<T>* v = Mlev + (size_t)sb * 4 * Kc;
          for (int n = 0; n <= P; ++n) {
            const int nk = n + kk;
            const int bi = nk * nk + nk + ll;
            {
              const Cx<T> ip = It[bi];
              for (int d = 0; d < 4; ++d) cfma(pt[d], v[d], ip);
              v += 4;
            }
            int m = 1;
            for (; m + 1 <= n; m += 2, v += 8) {
              pair(v, bi + m, bi - m, T(-1));
              pair(v + 4, bi + m + 1, bi - m - 1, T(1));
            }
            if (m <= n) {
              pair(v, bi + m, bi - m, T(-1));
              v += 4;
            }
          }
          // psi about the target centre: T(psi) - a . T(phi), a = c_t - c_s
          const T ax = (T)(vx * w), ay = (T)(vy * w), az = (T)(vz * w);
          pt[3].re -= ax * pt[0].re + ay * pt[1].re + az * pt[2].re;
          pt[3].im -= ax * pt[0].im + ay * pt[1].im + az * pt[2].im;
          for (int d = 0; d < 4; ++d) {
            acc[d].re = fma(sk_sign, pt[d].re, acc[d].re);
            acc[d].im = fma(sk_sign, pt[d].im, acc[d].im);
          }
        }
      }
  if (act) {
    Cx<T>* out = Lexp + (lv.off[lev] + (size_t)b) * 4 * Kc + (size_t)c * 4;
    for (int d = 0; d < 4; ++d) out[d] = acc[d];
  }
}

// Locals of level lev (side nl, width w) += the parent's locals translated to the box
// centre (L2L); the psi expansion moves from the parent centre to the child's by
// - (c' - c) . phi.  One workgroup per box, one thread per coefficient, four densities.
template <typename T>
__global__ void __launch_bounds__(256) k_fmm_l2l(int P, int nl, double w, const int* __restrict__ cnt,
                                                 const Cx<T>* __restrict__ tabR, const Cx<T>* __restrict__ Lpar,
                                                 Cx<T>* __restrict__ Llev) {
  __shared__ Cx<T> Ps[4][kFmmKc];
  __shared__ Cx<T> Rt[kFmmKc];
  const int b = blockIdx.x;
  if (cnt[b] == 0) return;
  const int Kc = tri(P + 1, 0);
  const int i = b % nl, j = (b / nl) % nl, k = b / (nl * nl);
  const int c = threadIdx.x;
  const bool act = c < Kc;
  int kk = 0, ll = 0;
  if (act) tri_inv(c, kk, ll);
  const int np = nl / 2;
  const int e = (i & 1) | ((j & 1) << 1) | ((k & 1) << 2);
  const T tx = (T)(((e & 1) - 0.5) * w), ty = (T)((((e >> 1) & 1) - 0.5) * w), tz = (T)(((e >> 2) - 0.5) * w);
  const Cx<T>* src = Lpar + (size_t)(((k / 2) * np + j / 2) * np + i / 2) * 4 * Kc;
  for (int q = threadIdx.x; q < Kc; q += blockDim.x) {
    const Cx<T> a = src[4 * q], bb = src[4 * q + 1], cc = src[4 * q + 2], dd = src[4 * q + 3];
    Ps[0][q] = a;
    Ps[1][q] = bb;
    Ps[2][q] = cc;
    Ps[3][q] = Cx<T>{dd.re - tx * a.re - ty * bb.re - tz * cc.re, dd.im - tx * a.im - ty * bb.im - tz * cc.im};
    Rt[q] = tabR[(size_t)e * Kc + q];
  }
  __syncthreads();
  if (!act) return;
  Cx<T>* out = Llev + ((size_t)b * Kc + c) * 4;
  Cx<T> acc[4];
  for (int d = 0; d < 4; ++d) acc[d] = out[d];
  for (int n = kk; n <= P; ++n)
    for (int l = max(-n, ll - (n - kk)); l <= min(n, ll + (n - kk)); ++l) {
      const Cx<T> r = cget(Rt, n - kk, l - ll);
      for (int d = 0; d < 4; ++d) cfma(acc[d], cget(Ps[d], n, l), r);
    }
  for (int d = 0; d < 4; ++d) out[d] = acc[d];
}

// Work items of the leaf kernel: (leaf, first target) for every 64 targets of a leaf.
__global__ void k_fmm_task_count(int nbox, const int* __restrict__ cnt, int* __restrict__ tcnt) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nbox) tcnt[b] = (cnt[b] + 63) / 64;
}

__global__ void k_fmm_task_fill(int nbox, const int* __restrict__ tcnt, const int* __restrict__ toff,
                                int2* __restrict__ task) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbox) return;
  for (int j = 0; j < tcnt[b]; ++j) task[toff[b] + j] = make_int2(b, 64 * j);
}

// Sources in leaf order: srt[p] = src[perm[p]] with the body index in v[6] and, in v[7], the
// body index that the four points from p on share, or -1.
template <typename T>
__global__ void k_fmm_pack_sorted(int N, const int* __restrict__ perm, const double4* __restrict__ Xs,
                                  const Src8<T>* __restrict__ src, Src8<T>* __restrict__ srt) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  Src8<T> s = src[perm[p]];
  const double body = Xs[p].w;
  bool one = p + 3 < N;
  for (int k = 1; k < 4; ++k) one = one && Xs[min(p + k, N - 1)].w == body;
  s.v[6] = (T)body;
  s.v[7] = one ? (T)body : T(-1);
  srt[p] = s;
}

// Leaf evaluation, one workgroup per work item (64 targets of one leaf, one per lane): far field
// from the leaf's local expansions, plus the direct traction sum over the points of the 27
// adjacent leaves that belong to other bodies.  The leaf is wave-uniform, so its expansion
// coefficients and the sources (9 contiguous ranges of the leaf-ordered points) are read
// with scalar loads.  Writes -(3/4pi)-scaled sums to out[3][N] at the original indices.
// The workgroup's waves take equal parts of the sources (the first, which also evaluates the
// expansions, as many fewer as that costs) and add their sums through LDS, in order: with a wave
// per work item the last wave of a CU ran alone for up to a third of the time, and small trees
// left SIMDs without one.
// Bound: the vector units, 21 operations a pair (26 with the mask of the same body's pairs on every
// pair).  1,248,000 points in 4096 leaves (9.3e9 pairs), float32: 5.68 -> 5.10 ms; the whole
// far_traction_fmm of 142,877 points 3.20 -> 2.62 ms.
template <typename T>
__global__ void __launch_bounds__(1024) k_fmm_leaf(int P, int nb, double lox, double loy, double loz, double w,
                                                  int N, const int2* __restrict__ task,
                                                  const int* __restrict__ start, const int* __restrict__ perm,
                                                  const double4* __restrict__ Xs, const double4* __restrict__ Ns,
                                                  const Src8<T>* __restrict__ srt, const Cx<T>* __restrict__ Lleaf,
                                                  int far_on, double* __restrict__ out) {
  extern __shared__ __align__(8) unsigned char leaf_lds[];
  T(*sum)[3][64] = reinterpret_cast<T(*)[3][64]>(leaf_lds);  // of the waves after the first
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const int2 tk = task[blockIdx.x];
  const int b = __builtin_amdgcn_readfirstlane(tk.x), t0 = __builtin_amdgcn_readfirstlane(tk.y);
  const int s0 = start[b], nt = start[b + 1] - s0;
  const int t = t0 + lane;
  const bool live = t < nt;
  const int Kc = tri(P + 1, 0);
  const int i = b % nb, j = (b / nb) % nb, k = b / (nb * nb);
  const double cx = lox + (i + 0.5) * w, cy = loy + (j + 0.5) * w, cz = loz + (k + 0.5) * w;
  const double4 xt = Xs[s0 + (live ? t : 0)], nn = Ns[s0 + (live ? t : 0)];
  const T xa = (T)xt.x, ya = (T)xt.y, za = (T)xt.z, nx = (T)nn.x, ny = (T)nn.y, nz = (T)nn.z;
  const T bt = (T)xt.w;
  T fx = 0, fy = 0, fz = 0;
  if (far_on && wv == 0) {
    const Cx<T>* Lb = Lleaf + (size_t)b * 4 * Kc;
    const T ssx = (T)(xt.x - cx), ssy = (T)(xt.y - cy), ssz = (T)(xt.z - cz);
    const T r2 = ssx * ssx + ssy * ssy + ssz * ssz;
    // gradient sums (d/dx + i d/dy) phi_0, phi_1 and d/dz phi_2; for all four densities
    // A = (d/dx + i d/dy)^2, B = d/dz (d/dx + i d/dy), C = d^2/dz^2
    Cx<T> g0{0, 0}, g1{0, 0}, g2{0, 0}, A[4], B[4], C[4];
    for (int dd = 0; dd < 4; ++dd) A[dd] = B[dd] = C[dd] = Cx<T>{0, 0};
    auto term = [&](int kk, int l, Cx<T> v) {
      if (kk <= P - 1) {
        cfma(g0, cget4(Lb, kk + 1, l + 1, 0), v);
        cfma(g1, cget4(Lb, kk + 1, l + 1, 1), v);
        cfma(g2, cget4(Lb, kk + 1, l, 2), v);
      }
      if (kk <= P - 2)
        for (int dd = 0; dd < 4; ++dd) {
          cfma(A[dd], cget4(Lb, kk + 2, l + 2, dd), v);
          cfma(B[dd], cget4(Lb, kk + 2, l + 1, dd), v);
          cfma(C[dd], cget4(Lb, kk + 2, l, dd), v);
        }
    };
    // R_kk^l(s) column by column (l >= 0): conj(R^l) for +l and (-1)^l R^l for -l
    T dre = 1, dim = 0;
    for (int l = 0; l <= P - 1; ++l) {
      if (l > 0) {
        const T inv = T(1) / T(2 * l);
        const T nre = (dre * ssx - dim * ssy) * inv, nim = (dre * ssy + dim * ssx) * inv;
        dre = nre;
        dim = nim;
      }
      T are = 0, aim = 0, bre = dre, bim = dim;
      for (int kk = l; kk <= P - 1; ++kk) {
        if (kk > l) {
          const T c1 = T(2 * kk - 1), inv = T(1) / T((kk - l) * (kk + l));
          const T vre = (c1 * ssz * bre - r2 * are) * inv, vim = (c1 * ssz * bim - r2 * aim) * inv;
          are = bre; aim = bim;
          bre = vre; bim = vim;
        }
        term(kk, l, Cx<T>{bre, -bim});
        if (l > 0) term(kk, -l, (l & 1) ? Cx<T>{-bre, -bim} : Cx<T>{bre, bim});
      }
    }
    const T div = g0.re + g1.im + g2.re;
    T H[4][6];  // xx, yy, zz, xy, xz, yz
    for (int dd = 0; dd < 4; ++dd) {
      H[dd][0] = T(0.5) * (A[dd].re - C[dd].re);
      H[dd][1] = T(0.5) * (-A[dd].re - C[dd].re);
      H[dd][2] = C[dd].re;
      H[dd][3] = T(0.5) * A[dd].im;
      H[dd][4] = B[dd].re;
      H[dd][5] = B[dd].im;
    }
    T Hs[6];
    for (int e = 0; e < 6; ++e) Hs[e] = H[3][e] - ssx * H[0][e] - ssy * H[1][e] - ssz * H[2][e];
    // the direct sum is kept in units of -(3/4pi): scale the far part by -(1/3)
    const T sc = T(-1.0 / 3.0);
    fx = sc * (div * nx + Hs[0] * nx + Hs[3] * ny + Hs[4] * nz);
    fy = sc * (div * ny + Hs[3] * nx + Hs[1] * ny + Hs[5] * nz);
    fz = sc * (div * nz + Hs[4] * nx + Hs[5] * ny + Hs[2] * nz);
  }
  // near field: traction of the other bodies' points in the 27 adjacent leaves.  Four sources per
  // step, their scalar loads issued a step ahead; if they are points of one body that no lane's
  // target belongs to, which is nearly always so, the pairs need no mask.  Otherwise
  // same-body pairs get weight 0, and |d|^2 + 1 keeps the point's own pair finite.
  auto near = [&](const Src8<T>& s, auto masked) {
    const T dx = xa - s.v[0], dy = ya - s.v[1], dz = za - s.v[2];
    T r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const T dn = dx * nx + dy * ny + dz * nz;
    const T dq = dx * s.v[3] + dy * s.v[4] + dz * s.v[5];
    T c = dn * dq;
    if (decltype(masked)::value && s.v[6] == bt) {
      r2 += T(1);
      c = T(0);
    }
    const T f = c * rinv5_t(r2);
    fx += f * dx;
    fy += f * dy;
    fz += f * dz;
  };
  // for each (nk, nj) the leaves ni - 1 .. ni + 1 are consecutive in leaf order
  const int i0 = max(0, i - 1), i1 = min(nb - 1, i + 1);
  const int k0 = max(0, k - 1), k1 = min(nb - 1, k + 1), j0 = max(0, j - 1), j1 = min(nb - 1, j + 1);
  int total = 0;
  for (int nk = k0; nk <= k1; ++nk)
    for (int nj = j0; nj <= j1; ++nj) {
      const int row = (nk * nb + nj) * nb;
      total += start[row + i1 + 1] - start[row + i0];
    }
  // this wave's part [from, to) of the concatenated ranges
  const int far = far_on ? fmm_far_cost(P) : 0, each = (total + far + nw - 1) / nw;
  const int from = __builtin_amdgcn_readfirstlane(max(0, wv * each - far));
  const int to = __builtin_amdgcn_readfirstlane(min(total, max(0, (wv + 1) * each - far)));
  int before = 0;
  for (int nk = k0; nk <= k1; ++nk)
    for (int nj = j0; nj <= j1; ++nj) {
      const int row = (nk * nb + nj) * nb;
      const int a0 = __builtin_amdgcn_readfirstlane(start[row + i0]);
      const int a1 = __builtin_amdgcn_readfirstlane(start[row + i1 + 1]);
      int q = a0 + max(0, from - before);
      const int e = min(a1, a0 + (to - before));
      before += a1 - a0;
      if (q + 4 <= e) {
        Src8<T> n0 = srt[q], n1 = srt[q + 1], n2 = srt[q + 2], n3 = srt[q + 3];
        for (; q + 4 <= e; q += 4) {
          const Src8<T> s0 = n0, s1 = n1, s2 = n2, s3 = n3;
          const int nq = min(q + 4, e - 4);
          n0 = srt[nq];
          n1 = srt[nq + 1];
          n2 = srt[nq + 2];
          n3 = srt[nq + 3];
          if (!__any(s0.v[7] < T(0) || s0.v[7] == bt)) {
            near(s0, std::false_type{});
            near(s1, std::false_type{});
            near(s2, std::false_type{});
            near(s3, std::false_type{});
          } else {
            near(s0, std::true_type{});
            near(s1, std::true_type{});
            near(s2, std::true_type{});
            near(s3, std::true_type{});
          }
        }
      }
      for (; q < e; ++q) near(srt[q], std::true_type{});
    }
  if (wv > 0) {
    sum[wv - 1][0][lane] = fx;
    sum[wv - 1][1][lane] = fy;
    sum[wv - 1][2][lane] = fz;
  }
  __syncthreads();
  if (wv > 0) return;
  for (int v = 0; v < nw - 1; ++v) {
    fx += sum[v][0][lane];
    fy += sum[v][1][lane];
    fz += sum[v][2][lane];
  }
  if (live) {
    const int g = perm[s0 + t];
    const double sc = -3.0 / (4.0 * RBM_PI);
    out[g] = sc * (double)fx;
    out[(size_t)N + g] = sc * (double)fy;
    out[2 * (size_t)N + g] = sc * (double)fz;
  }
}

// ---------------------------------------------------------------------------------
// Launchers

hipError_t launch_fmm_bounds(int N, const double* X, double* scratch, double* out6, hipStream_t st) {
  const int nwg = std::min(512, (N + 1023) / 1024);
  if (nwg == 1) {
    k_fmm_bounds<true><<<1, 256, 0, st>>>(N, X, out6);
  } else {
    k_fmm_bounds<true><<<nwg, 256, 0, st>>>(N, X, scratch);
    k_fmm_bounds<false><<<1, 256, 0, st>>>(nwg, scratch, out6);
  }
  return hipGetLastError();
}

hipError_t launch_fmm_sort_points(int N, int M, const double* X, const double* Nn, const double* lo, double w,
                                  int nb, int* leaf, int* cnt, int* start, int* fill, int* perm, int* maxcnt,
                                  double4* Xs, double4* Ns, hipStream_t st) {
  const int nbox = nb * nb * nb;
  hipError_t e;
  if ((e = hipMemsetAsync(cnt, 0, (size_t)nbox * sizeof(int), st)) != hipSuccess) return e;
  if ((e = hipMemsetAsync(fill, 0, (size_t)nbox * sizeof(int), st)) != hipSuccess) return e;
  k_fmm_count<<<(N + 255) / 256, 256, 0, st>>>(N, X, lo[0], lo[1], lo[2], w, nb, leaf, cnt);
  k_fmm_scan<<<1, 1024, 0, st>>>(nbox, cnt, start, maxcnt);
  k_fmm_scatter<<<(N + 255) / 256, 256, 0, st>>>(N, leaf, start, fill, perm);
  return hipGetLastError();
}

hipError_t launch_fmm_finish_tree(int N, int M, int L, const double* X, const double* Nn, const int* start,
                                  int* perm, double4* Xs, double4* Ns, int* const* cnt_lev, int* tcnt, int* toff,
                                  int2* task, int* scratch, hipStream_t st) {
  const int nb = 1 << L, nbox = nb * nb * nb;
  k_fmm_sort<<<nbox, 256, 0, st>>>(start, perm);
  k_fmm_gather<<<(N + 255) / 256, 256, 0, st>>>(N, M, perm, X, Nn, Xs, Ns);
  for (int lev = L - 1; lev >= 2; --lev) {
    const int np = 1 << lev;
    k_fmm_level_count<<<(np * np * np + 255) / 256, 256, 0, st>>>(np, cnt_lev[lev + 1], cnt_lev[lev]);
  }
  k_fmm_task_count<<<(nbox + 255) / 256, 256, 0, st>>>(nbox, cnt_lev[L], tcnt);
  k_fmm_scan<<<1, 1024, 0, st>>>(nbox, tcnt, toff, scratch);
  k_fmm_task_fill<<<(nbox + 255) / 256, 256, 0, st>>>(nbox, tcnt, toff, task);
  return hipGetLastError();
}

static int fmm_threads(int P) {
  const int o = 4 * tri(P + 1, 0);
  return (o + 63) / 64 * 64;
}

// Translations by rotation or dense.  At order 12 and 4096 leaves the dense kernel takes 5.1 ms, the
// rotations 1.45; they have float32 tables, and two tiles of 8 orders each.
template <typename T>
static constexpr bool fmm_rotates(int P) { return sizeof(T) == 4 && P <= kFmmRotOrder; }

template <typename T>
hipError_t launch_fmm_tables(int P, int L, double D, void* tabR, void* tabI, hipStream_t st) {
  if (P < 2 || P > kFmmPMax || L < 2) return hipErrorInvalidValue;
  const int nv = fmm_rotates<T>(P) ? 0 : kFmmVecs;
  dim3 grid((8 + nv + 63) / 64, L - 1);
  k_fmm_tables<T><<<grid, 64, 0, st>>>(P, L, D, nv, static_cast<Cx<T>*>(tabR), static_cast<Cx<T>*>(tabI));
  return hipGetLastError();
}

// One evaluation of the traction sums for the sources src (packed, original order):
// multipoles up, locals down, leaf evaluation into out[3][N].  Mexp/Lexp hold levels
// 2..L at box offsets lev_off[lev]; cnt_lev[lev] the points per box.
template <typename T>
hipError_t launch_fmm_apply(int P, int L, const double* lo, double D, int N, const int* start, const int* perm,
                            const double4* Xs, const double4* Ns, int* const* cnt_lev, const size_t* lev_off,
                            int ntask, const int2* task, const void* tabR, const void* tabI, int max_level,
                            const float* rot, const void* src, void* srt, void* Mexp, void* Lexp, double* out,
                            hipStream_t st) {
  if (P < 2 || P > kFmmPMax || L < 0) return hipErrorInvalidValue;
  const int nb = 1 << L, Kc = tri(P + 1, 0);
  const double w = ldexp(D, -L);
  Src8<T>* so = static_cast<Src8<T>*>(srt);
  Cx<T>* Mx = static_cast<Cx<T>*>(Mexp);
  Cx<T>* Lx = static_cast<Cx<T>*>(Lexp);
  const Cx<T>* tR = static_cast<const Cx<T>*>(tabR);
  const Cx<T>* tI = static_cast<const Cx<T>*>(tabI);
  const int th = fmm_threads(P);
  const bool far_on = L >= 2;
  k_fmm_pack_sorted<T><<<(N + 255) / 256, 256, 0, st>>>(N, perm, Xs, static_cast<const Src8<T>*>(src), so);
  if (far_on) {
    k_fmm_p2m<T><<<nb * nb * nb, th, 0, st>>>(P, nb, lo[0], lo[1], lo[2], w, start, perm, Xs, so,
                                              Mx + lev_off[L] * 4 * Kc);
    for (int lev = L; lev > 2; --lev) {
      const int nc = 1 << lev, np = nc / 2;
      k_fmm_m2m<T><<<np * np * np, th, 0, st>>>(P, nc, ldexp(D, -lev), cnt_lev[lev],
                                                tR + (size_t)(lev - 2) * 8 * Kc, Mx + lev_off[lev] * 4 * Kc,
                                                Mx + lev_off[lev - 1] * 4 * Kc);
    }
    if (L > 6) return hipErrorInvalidValue;
    FmmLevels lv{};
    int nwg = 0;
    for (int lev = 2; lev <= L; ++lev) {
      lv.cnt[lev] = cnt_lev[lev];
      lv.off[lev] = lev_off[lev];
      lv.first[lev] = nwg;
      nwg += 1 << (3 * lev);
    }
    lv.first[L + 1] = nwg;
    const int thl = (Kc + 63) / 64 * 64;
    bool done = false;
    if constexpr (sizeof(T) == 4) {
      if (fmm_rotates<T>(P)) {
        const hipError_t e = launch_fmm_m2l_rot(P, L, max_level, D, lv, rot, Mx, Lx, st);
        if (e != hipSuccess) return e;
        done = true;
      }
    }
    if (!done) k_fmm_m2l<T><<<nwg, thl, 0, st>>>(P, L, D, lv, tI, Mx, Lx);
    for (int lev = 3; lev <= L; ++lev) {
      const int nl = 1 << lev;
      k_fmm_l2l<T><<<nl * nl * nl, thl, 0, st>>>(P, nl, ldexp(D, -lev), cnt_lev[lev], tR + (size_t)(lev - 2) * 8 * Kc,
                                                Lx + lev_off[lev - 1] * 4 * Kc, Lx + lev_off[lev] * 4 * Kc);
    }
  }
  const int nw = fmm_leaf_waves(N, ntask, nb * nb * nb, P, far_on);
  if (ntask > 0)
    k_fmm_leaf<T><<<ntask, 64 * nw, (nw - 1) * 3 * 64 * sizeof(T), st>>>(P, nb, lo[0], lo[1], lo[2], w, N, task, start, perm, Xs,
                                                   Ns, so, far_on ? Lx + lev_off[L] * 4 * Kc : nullptr,
                                                   far_on ? 1 : 0, out);
  return hipGetLastError();
}

template hipError_t launch_fmm_tables<double>(int, int, double, void*, void*, hipStream_t);
template hipError_t launch_fmm_tables<float>(int, int, double, void*, void*, hipStream_t);
template hipError_t launch_fmm_apply<double>(int, int, const double*, double, int, const int*, const int*,
                                             const double4*, const double4*, int* const*, const size_t*, int,
                                             const int2*, const void*, const void*, int, const float*,
                                             const void*, void*, void*, void*, double*, hipStream_t);
template hipError_t launch_fmm_apply<float>(int, int, const double*, double, int, const int*, const int*,
                                            const double4*, const double4*, int* const*, const size_t*, int,
                                            const int2*, const void*, const void*, int, const float*, const void*,
                                            void*, void*, void*, double*, hipStream_t);

}  // namespace rbm
