// Singular self operators by grid rotation (§3 and the rule of Gimbutas-Veerapaneni cited
// there), float64.  For the rotated nodes s_q = Q_t s'_q, Q_t = R_z(phi_t) R_y(theta_t):
//   C[k][b] = sum_q W_q J(s_q) kern_k(x_t, x(s_q)) Y_b(s_q)         (b in B_p)
//   row(t)  = C F                                                     (F: grid -> B_p)
// kern = Stokeslet/eta (S) and n_t . T (K); both 3x3 symmetric (6 entries each).
//
// Everything is done in the rotated frame, where the nodes s' are a grid of Gauss-Legendre
// colatitudes times uniform azimuths and sums over them separate:
//   1. the surface's coefficients rotated into the frame: by R_z a mixing of +-m, by R_y the
//      matrices D_l(theta_t), which couple cosines with cosines and sines with sines only;
//   2. x - x_t, x_theta, x_phi / sin(theta) on the grid: a sum over l per (colatitude, m), then the
//      sum over m, whose cosine and sine parts give the azimuths phi and -phi together
//      (J = |x_theta x x_phi / sin| does not depend on the orthonormal frame it is taken in);
//   3. the kernels at the nodes; their sums and differences over +-phi against cos(m phi) and
//      sin(m phi), then the sum over colatitudes per (l, m): C in the rotated frame;
//   4. C rotated back by D_l; the rotation by R_z only shifts the azimuths of the grid F is
//      evaluated on: the sum over l per (grid colatitude, m), then over m.
// About 0.9 million multiply-adds per target at p = 12 instead of the 4.9 million of tabulating the
// harmonics at every rotated node and contracting with them, and no Legendre sweep per node.
// The two sums over azimuths (2 and 3) are products on the float64 matrix cores.
// Bound: latency.  Two workgroups a CU (registers: E and O of step 2), each a chain of short
// phases between barriers; vector units about 40%, matrix cores 17% busy.
// 64 shapes at p = 12, p_sing = 24: 20.5 -> 2.13 ms + 0.05 ms of tables; setup of them
// 30.8 -> 12.7 ms, of 35 shapes at p = 16 339 -> 42 ms, of 8 at p = 11 6.1 -> 4.1 ms.
//
// S and K are written row-major in the body frame, entry (row = c*M + t, col = c'*M + a) at
// [row*3M + col]: a workgroup holds one target's rows, so these stores run along the rows.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "pair.h"

namespace rbm {

// Places of the tables in one buffer (doubles).  NIP colatitudes and azimuths padded to 32, m
// padded to a multiple of 16; padding holds zeros.
struct SingularTables {
  int p, ps, NIP, MP;
  size_t lg, lt, tc, ts, dw, gg, total;
};

__host__ __device__ inline int rot_offset(int l) { return l * (2 * l * l + 1) / 3; }  // of D_l: sum of (k+1)^2 + k^2

static SingularTables singular_tables(int p, int ps) {
  SingularTables t;
  t.p = p;
  t.ps = ps;
  t.NIP = (ps + 1 + 31) / 32 * 32;
  t.MP = (p + 1 + 15) / 16 * 16;
  const size_t nc = (size_t)(p + 1) * (p + 1);
  size_t o = 0;
  auto take = [&](size_t n) { const size_t at = o; o += (n + 31) / 32 * 32; return at; };
  t.lg = take(3 * (size_t)t.MP * (p + 1) * t.NIP);  // [P, D, mQ][m][l - m][i], sqrt2 included for m > 0
  t.lt = take((size_t)t.NIP * nc);                   // [i][l^2 + l + m] P
  t.tc = take((size_t)t.MP * t.NIP);                 // [m][n] cos(m phi'_n), n <= ps
  t.ts = take((size_t)t.MP * t.NIP);
  t.dw = take((size_t)(p + 1) * rot_offset(p + 1));  // [j] D_l(theta_j)
  t.gg = take((p + 1) * nc);                         // [j][l^2 + l + m] forward transform, no azimuths
  t.total = o;
  return t;
}

size_t singular_table_doubles(int p, int ps) { return singular_tables(p, ps).total; }

// Double-double arithmetic (an unevaluated sum hi + lo, Dekker's and Knuth's error-free sums and
// fma products) for the tables: the recurrences lose about a digit by degree 20, and an error of a
// table entry, unlike the rounding of a sum over nodes, is common to all targets and nodes.
// In plain float64 they gave 110 eps of the incident field on a sphere at p = 20 instead of 73.
struct dd {
  double hi, lo;
};
__device__ __forceinline__ dd quick_two(double a, double b) {
  const double s = a + b;
  return {s, b - (s - a)};
}
__device__ __forceinline__ dd two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
__device__ __forceinline__ dd operator+(dd a, dd b) {
  const dd s = two_sum(a.hi, b.hi), t = two_sum(a.lo, b.lo);
  const dd u = quick_two(s.hi, s.lo + t.hi);
  return quick_two(u.hi, u.lo + t.lo);
}
__device__ __forceinline__ dd operator-(dd a) { return {-a.hi, -a.lo}; }
__device__ __forceinline__ dd operator-(dd a, dd b) { return a + -b; }
__device__ __forceinline__ dd operator*(dd a, dd b) {
  const double h = a.hi * b.hi;
  return quick_two(h, fma(a.hi, b.hi, -h) + (a.hi * b.lo + a.lo * b.hi));
}
__device__ __forceinline__ dd operator*(double a, dd b) { return dd{a, 0.0} * b; }
__device__ __forceinline__ dd operator/(dd a, dd b) {
  const double q = a.hi / b.hi;
  const dd r = a - q * b;
  return quick_two(q, r.hi / b.hi);
}
__device__ __forceinline__ dd sqrt_dd(dd a) {
  if (!(a.hi > 0.0)) return {0.0, 0.0};
  const double y = sqrt(a.hi);
  const dd r = a - dd{y, 0.0} * dd{y, 0.0};
  return quick_two(y, r.hi / (2.0 * y));
}
__device__ __forceinline__ dd sqrt_dd(double a) { return sqrt_dd(dd{a, 0.0}); }
__device__ __forceinline__ dd sin_of(double x) {  // sqrt(1 - x^2)
  return sqrt_dd(two_sum(1.0, -x) * two_sum(1.0, x));
}

// d^l_{M,M'}(theta) by the recurrence in l from l = max(M, |M'|), with c = cos(theta/2) and
// s = sin(theta/2).  M >= 0.
struct WignerChain {
  int l, M, Mp;
  double ct, q0;  // q0: (l^2 - M^2)(l^2 - M'^2)
  dd v, prev;
  __device__ __forceinline__ WignerChain(int M_, int Mp_, double ct_, dd c, dd s) : M(M_), Mp(Mp_), ct(ct_) {
    l = max(M, abs(Mp));
    const int ec = abs(M + Mp), es = abs(M - Mp);
    double binom = 1.0;  // (2l over ec), at most (40 over 20): exact
    for (int k = 1; k <= ec; ++k) binom = binom * (2 * l - ec + k) / k;
    v = sqrt_dd(binom);
    for (int k = 0; k < ec; ++k) v = v * c;
    for (int k = 0; k < es; ++k) v = v * s;
    if (Mp > M && (es & 1)) v = -v;
    prev = {0.0, 0.0};
    q0 = 0.0;
  }
  __device__ __forceinline__ void step() {
    const double l1 = l + 1.0, q1 = (l1 * l1 - (double)(M * M)) * (l1 * l1 - (double)(Mp * Mp));
    const dd next = l == 0 ? ct * v
                           : ((2.0 * l + 1.0) * (((l * l1) * dd{ct, 0.0} - dd{(double)(M * Mp), 0.0}) * v) -
                              l1 * (sqrt_dd(q0) * prev)) / ((double)l * sqrt_dd(q1));
    prev = v;
    v = next;
    q0 = q1;
    ++l;
  }
};

// D_l(theta_j)[m][m'] with Y_lm(R_y(theta_j) s) = sum_m' D[m][m'] Y_lm'(s): cosines m, m' = 0..l,
// d_{m,m'} + (-1)^m' d_{m,-m'} (over sqrt 2 for m = 0 and for m' = 0), then sines m, m' = 1..l, the same
// with minus.  One thread per (m, m', j).
__global__ __launch_bounds__(64) void k_rotation_matrices(int p, const double* __restrict__ glt,
                                                          double* __restrict__ dw) {
  const int e = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y;
  if (e >= (p + 1) * (p + 1)) return;
  const int m = e / (p + 1), mp = e % (p + 1);
  const double ct = glt[j];
  const dd c = sqrt_dd(0.5 * two_sum(1.0, ct)), s = sqrt_dd(0.5 * two_sum(1.0, -ct));
  const dd half = {0.5, 0.0}, h = {0.7071067811865476, -4.833646656726457e-17};  // 1 / sqrt 2
  const dd f = m == 0 && mp == 0 ? half : m == 0 || mp == 0 ? h : dd{1.0, 0.0};
  double* D = dw + (size_t)j * rot_offset(p + 1);
  WignerChain x(m, mp, ct, c, s), y(m, -mp, ct, c, s);
  for (int l = x.l;; ++l) {
    const dd b = mp & 1 ? -y.v : y.v;
    D[rot_offset(l) + m * (l + 1) + mp] = (f * (x.v + b)).hi;
    if (m > 0 && mp > 0) D[rot_offset(l) + (l + 1) * (l + 1) + (m - 1) * l + mp - 1] = (x.v - b).hi;
    if (l == p) break;
    x.step();
    y.step();
  }
}

// Legendre tables at the rotated colatitudes, a thread per (colatitude, m), the recurrences of
// legendre_sweep in double-double; the grid's (last block); the azimuth tables.
__global__ __launch_bounds__(64) void k_singular_tables(SingularTables t, const double* __restrict__ glr_t,
                                                        const double* __restrict__ glt,
                                                        const double* __restrict__ glw, double* __restrict__ tab) {
  const int p = t.p, nc = (p + 1) * (p + 1), nb = t.NIP * t.MP / 64;
  if ((int)blockIdx.x < nb) {
    const int e = blockIdx.x * 64 + threadIdx.x, i = e % t.NIP, m = e / t.NIP;
    const bool live = i <= t.ps && m <= p;
    const size_t plane = (size_t)t.MP * (p + 1) * t.NIP;
    double* o = tab + t.lg + (size_t)m * (p + 1) * t.NIP + i;
    double* ol = tab + t.lt + (size_t)i * nc;
    const dd zero = {0.0, 0.0}, y00 = {0.28209479177387814, 3.83386490329147e-18};  // 1 / sqrt(4 pi)
    // The plane of P gives the positions, taken relative to the target at the pole of the frame: P_l0 less
    // its value there, formed before it is rounded.  The difference of two rounded positions loses digits
    // at the nodes next to the target, where the kernels are largest: rounding errors of K at p = 6, 12, 14 and
    // 20 against long double 2.2, 3.2, 3.0 and 3.2 eps of its largest entry (rms), with this 0.8, 0.8, 0.4 and 1.5.
    auto put = [&](int l, dd P, dd Q, dd D) {
      const size_t at = (size_t)(l - m) * t.NIP;
      o[at] = m == 0 && live ? (P - sqrt_dd(2.0 * l + 1.0) * y00).hi : P.hi;
      o[at + plane] = D.hi;
      o[at + 2 * plane] = ((double)m * Q).hi;
      if (m > p) return;
      ol[l * l + l + m] = P.hi;
      ol[l * l + l - m] = P.hi;
    };
    int l = m;
    if (live) {
      const double x = glr_t[i];
      const dd s = sin_of(x), r2 = {1.4142135623730951, -9.667293313452913e-17};  // sqrt 2
      dd p0 = y00, q0 = zero;
      if (m) p0 = r2 * p0;
      for (int k = 1; k <= m; ++k) {
        q0 = sqrt_dd(dd{2.0 * k + 1.0, 0.0} / dd{2.0 * k, 0.0}) * p0;
        p0 = s * q0;
      }
      dd d0 = x * ((double)m * q0), p1 = zero, q1 = zero, d1 = zero;
      put(l++, p0, q0, d0);
      if (l <= p) {
        const dd c = sqrt_dd(2.0 * m + 3.0);
        p1 = c * (x * p0);
        q1 = c * (x * q0);
        d1 = c * (x * d0 - s * p0);
        put(l++, p1, q1, d1);
      }
      for (; l <= p; ++l) {
        const double ll = (double)l * l, k2 = (l - 1.0) * (l - 1.0), m2 = (double)m * m;
        const dd a = sqrt_dd(dd{4.0 * ll - 1.0, 0.0} / dd{ll - m2, 0.0});
        const dd b = sqrt_dd(dd{k2 - m2, 0.0} / dd{4.0 * k2 - 1.0, 0.0});
        const dd p2 = a * (x * p1 - b * p0), q2 = a * (x * q1 - b * q0), d2 = a * (x * d1 - s * p1 - b * d0);
        put(l, p2, q2, d2);
        p0 = p1; p1 = p2; q0 = q1; q1 = q2; d0 = d1; d1 = d2;
      }
    }
    for (; l <= p; ++l) put(l, zero, zero, zero);
    // places of this row of m beyond its degrees (all of them for m > p)
    for (int d = max(0, p - m + 1); d <= p; ++d)
      for (int k = 0; k < 3; ++k) o[(size_t)d * t.NIP + k * plane] = 0.0;
    double sn = 0.0, cs = 0.0;
    if (live) sincospi((double)m * i / t.ps, &sn, &cs);
    tab[t.tc + (size_t)m * t.NIP + i] = cs;
    tab[t.ts + (size_t)m * t.NIP + i] = sn;
  } else {
    const double r2 = 1.41421356237309504880;
    const int j = threadIdx.x;
    if (j > p) return;
    const double x = glt[j], s = sqrt(fmax(0.0, 1.0 - x * x)), wq = RBM_PI / p * glw[j];
    legendre_sweep(p, x, s, [&](int l, int m, double P, double, double) {
      const double v = wq * P * (m ? r2 : 1.0) * (l == p && m == p ? 0.5 : 1.0);
      tab[t.gg + (size_t)j * nc + l * l + l + m] = v;
      tab[t.gg + (size_t)j * nc + l * l + l - m] = v;
    });
  }
}

typedef double d4s __attribute__((ext_vector_type(4)));

// LDS of k_singular in doubles: rotated coefficients, azimuth table, and the work area that
// holds in turn the node kernels of 8 colatitudes x 32 azimuths (sums and differences), their
// azimuthal sums, C in both frames and the colatitude sums of F.
constexpr int kKwRow = 34;                       // node kernels: row stride, free of bank conflicts where rows are read
constexpr int kKwSize = 2 * 96 * kKwRow;
__host__ __device__ inline int singular_work(int p) {
  const int nc = (p + 1) * (p + 1), cc = 24 * nc, ce = 12 * nc + 12 * (p + 1) * (2 * p + 1);
  int w = kKwSize > cc ? kKwSize : cc;
  return w > ce ? w : ce;
}

// One workgroup per (target, shape).  The sums and differences over +-n of 8 colatitudes at a time go
// through LDS (one e of the four rows a lane holds), so that two workgroups fit a CU.  NIT: passes
// of 256 threads over the (l, m) x 3 sums of step 3; MT: 16-wide tiles of m.
template <int NIT, int MT>
__global__ __launch_bounds__(256, NIT == 2 ? 2 : 1) void k_singular(
    SingularTables T, double eta, const double* __restrict__ coef_all, const double* __restrict__ gn_all,
    const double* __restrict__ rW, const double* __restrict__ tab, double* __restrict__ Sop, double* __restrict__ Kop) {
  extern __shared__ double lds[];
  const int p = T.p, ps = T.ps, NIP = T.NIP, nc = (p + 1) * (p + 1), M = (p + 1) * 2 * p, M3 = 3 * M;
  const int MQ = (p + 1 + 3) / 4 * 4, p1 = p + 1;
  const int t = blockIdx.x, s = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int jt = t / (2 * p), kt = t % (2 * p);
  double* cr = lds;                                // [3][cos, sin][MQ][p1 (l - m)] rotated coefficients
  double* az = cr + 6 * MQ * p1;                   // [cos, sin][2p] of pi r / p
  double* work = az + 4 * p;
  // 1. coefficients: R_z into `work`, then D
  for (int r = tid; r < 2 * p; r += 256) sincospi((double)r / p, &az[2 * p + r], &az[r]);
  for (int i = tid; i < 6 * MQ * p1; i += 256) cr[i] = 0.0;
  __syncthreads();
  const double* coef = coef_all + (size_t)s * 3 * nc;
  for (int e = tid; e < 3 * nc; e += 256) {
    const int c = e / nc, b = e % nc;
    int l = (int)sqrtf((float)b);
    l += (l + 1) * (l + 1) <= b;
    l -= l * l > b;
    const int m = b - l * l - l, am = m < 0 ? -m : m, r = (am * kt) % (2 * p);
    const double cp = coef[c * nc + l * l + l + am], cm = am ? coef[c * nc + l * l + l - am] : 0.0;
    work[e] = m >= 0 ? cp * az[r] + cm * az[2 * p + r] : cm * az[r] - cp * az[2 * p + r];
  }
  __syncthreads();
  const double* dw = tab + T.dw + (size_t)jt * rot_offset(p + 1);
  for (int b = tid; b < nc; b += 256) {
    int l = (int)sqrtf((float)b);
    l += (l + 1) * (l + 1) <= b;
    l -= l * l > b;
    const int mp = b - l * l - l, odd = mp < 0, am = odd ? -mp : mp;
    const double* z = work + l * l + l;
    const double* D = dw + rot_offset(l) + (odd ? (l + 1) * (l + 1) + am - 1 : am);
    const int dd = odd ? l : l + 1, sg = odd ? -1 : 1;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
    for (int m = odd; m <= l; ++m, D += dd)
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = fma(z[c * nc + sg * m], *D, v[c]);
#pragma unroll
    for (int c = 0; c < 3; ++c) cr[((c * 2 + odd) * MQ + am) * p1 + l - am] = v[c];
  }
  __syncthreads();
  const double* gn = gn_all + (size_t)s * 3 * M;
  const double nt0 = gn[t], nt1 = gn[M + t], nt2 = gn[2 * M + t];
  const double cS = 1.0 / (8.0 * RBM_PI * eta), cK = 3.0 / (4.0 * RBM_PI);
  const double* LG = tab + T.lg;
  const size_t plane = (size_t)T.MP * p1 * NIP;
  const double* LT = tab + T.lt;
  const double* TC = tab + T.tc;
  const double* TS = tab + T.ts;
  double cacc[NIT][4];
#pragma unroll
  for (int u = 0; u < NIT; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) cacc[u][k] = 0.0;
  for (int ib = 0; ib <= ps; ib += 32)
    for (int nb = 0; nb <= ps; nb += 32) {
      // 2. this wave's 16 colatitudes x 16 azimuths: rows (lk + 4 e) of colatitudes, column lr
      const int i0 = ib + 16 * (wv >> 1), n0 = nb + 16 * (wv & 1);
      d4s E[9], O[9];
#pragma unroll
      for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) E[k][e] = O[k][e] = 0.0;
      for (int ks = 0; ks < MQ; ks += 4) {
        const int m = ks + lk;
        double ge[9], go[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) ge[k] = go[k] = 0.0;
        unsigned at = m * p1 * NIP + i0 + lr;
        const unsigned last = at + (p - ks) * NIP;
        const double* A = cr + m * p1;
        const double bc = TC[(size_t)m * NIP + n0 + lr], bs = TS[(size_t)m * NIP + n0 + lr];
        // four steps' table values in flight; the table's zeros end each row of m
        double nx[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int k = 0; k < 3; ++k) nx[q][k] = (LG + k * plane)[min(at + q * NIP, last)];
        at += 4 * NIP;
        for (int d0 = 0; d0 <= p - ks; d0 += 4) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int d = d0 + q;
            if (d > p - ks) break;
            const double P = nx[q][0], D = nx[q][1], Q = nx[q][2];
#pragma unroll
            for (int k = 0; k < 3; ++k) nx[q][k] = (LG + k * plane)[min(at, last)];
            at += NIP;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const double a = A[c * 2 * MQ * p1 + d], b = A[(c * 2 + 1) * MQ * p1 + d];
              ge[c] += a * P;
              go[c] += b * P;
              ge[3 + c] += a * D;
              go[3 + c] += b * D;
              ge[6 + c] += b * Q;
              go[6 + c] -= a * Q;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          E[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(ge[k], bc, E[k], 0, 0, 0);
          O[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(go[k], bs, O[k], 0, 0, 0);
        }
      }
      // cos and sin of the azimuths against m, this wave's half of the products of step 3
      double trig[MT][8];
      const double* TR = wv < 2 ? TC : TS;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < 8; ++q) trig[mt][q] = TR[(size_t)(16 * mt + lr) * NIP + nb + 4 * q + lk];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // 3. kernels at (i, +-n)
        const int i = i0 + lk + 4 * e, n = n0 + lr;
        const bool live = i <= ps && n <= ps, twice = n != 0 && n != ps;
        const double W = rW[(size_t)min(i, ps) * 2 * ps];
        // per sign: x - x_t and the weights of delta, r r (Stokeslet) and r r (traction)
        double r[2][3], wd[2], ws[2], wk[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          double v[9];
#pragma unroll
          for (int k = 0; k < 9; ++k) v[k] = g ? E[k][e] - O[k][e] : E[k][e] + O[k][e];
          const double c0 = v[4] * v[8] - v[5] * v[7], c1 = v[5] * v[6] - v[3] * v[8], c2 = v[3] * v[7] - v[4] * v[6];
          const double w = W * sqrt(c0 * c0 + c1 * c1 + c2 * c2);
          r[g][0] = v[0];
          r[g][1] = v[1];
          r[g][2] = v[2];
          const double di = rsqrt_t(r[g][0] * r[g][0] + r[g][1] * r[g][1] + r[g][2] * r[g][2]);
          const double di3 = di * di * di, rn = r[g][0] * nt0 + r[g][1] * nt1 + r[g][2] * nt2;
          const bool on = live && (g == 0 || twice);
          wd[g] = on ? w * cS * di : 0.0;
          ws[g] = on ? w * cS * di3 : 0.0;
          wk[g] = on ? w * cK * rn * di3 * di * di : 0.0;
        }
        double* o = work + (size_t)(12 * (4 * (wv >> 1) + lk)) * kKwRow + 16 * (wv & 1) + lr;
        const int ki[6] = {0, 1, 2, 0, 0, 1}, kj[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          const double q0 = r[0][ki[k]] * r[0][kj[k]], q1 = r[1][ki[k]] * r[1][kj[k]];
          const double s0 = fma(ws[0], q0, k < 3 ? wd[0] : 0.0), s1 = fma(ws[1], q1, k < 3 ? wd[1] : 0.0);
          const double t0 = wk[0] * q0, t1 = wk[1] * q1;
          o[k * kKwRow] = s0 + s1;
          o[(6 + k) * kKwRow] = t0 + t1;
          o[(96 + k) * kKwRow] = twice ? s0 - s1 : 0.0;
          o[(102 + k) * kKwRow] = twice ? t0 - t1 : 0.0;
        }
        __syncthreads();
        // this thread's Legendre values of the last step, on their way during the next
        // (the empty asm keeps their loads from being hoisted out of the loop over azimuths: 152
        // registers were spilled then at NIT = 2, 35 are now)
        double lw[2][8];
        auto load_lw = [&](int u) {
          unsigned at = (unsigned)min(tid + 256 * u, 3 * nc - 1) % (unsigned)nc;
          asm volatile("" : "+v"(at));
#pragma unroll
          for (int g = 0; g < 8; ++g)
            lw[u & 1][g] = (LT + (ib + 4 * e + 16 * (g >> 2) + (g & 3)) * nc)[at];
        };
        load_lw(0);
        // sums over 32 azimuths: 96 rows (colatitude, kernel) x m; waves 0, 1 the cosines of the
        // sums, waves 2, 3 the sines of the differences, three 16-row tiles each
        d4s h[3][MT];
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int k = 0; k < 4; ++k) h[u][mt][k] = 0.0;
        const int tile = (wv >> 1) * 96 + (wv & 1) * 48;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (q % 4 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            const double a = work[(tile + 16 * u + lr) * kKwRow + 4 * q + lk];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              h[u][mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, trig[mt][q], h[u][mt], 0, 0, 0);
          }
        }
        __syncthreads();
        constexpr int HR = 16 * MT + 1;
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int k = 0; k < 4; ++k) work[(tile + 16 * u + lk + 4 * k) * HR + 16 * mt + lr] = h[u][mt][k];
        __syncthreads();
        // sums over these eight colatitudes for every (l, m) and a third of the kernels
#pragma unroll
        for (int u = 0; u < NIT; ++u) {
          const int it = tid + 256 * u;
          if (u + 1 < NIT) load_lw(u + 1);
          if (it < 3 * nc) {
            const int b = it % nc, kg = it / nc;
            int l = (int)sqrtf((float)b);
            l += (l + 1) * (l + 1) <= b;
            l -= l * l > b;
            const int m = b - l * l - l;
            const double* hr = work + ((m < 0 ? 96 : 0) + 4 * kg) * HR + (m < 0 ? -m : m);
#pragma unroll
            for (int g = 0; g < 8; ++g)
#pragma unroll
              for (int k = 0; k < 4; ++k) cacc[u][k] += lw[u & 1][g] * hr[(12 * g + k) * HR];
          }
        }
        __syncthreads();
      }
    }
  // 4. C back from the rotated frame
  double* C1 = work;              // [12][nc]
  double* C2 = work + 12 * nc;    // [12][nc]
#pragma unroll
  for (int u = 0; u < NIT; ++u) {
    const int it = tid + 256 * u;
    if (it < 3 * nc)
#pragma unroll
      for (int k = 0; k < 4; ++k) C1[(4 * (it / nc) + k) * nc + it % nc] = cacc[u][k];
  }
  __syncthreads();
  for (int it = tid; it < 3 * nc; it += 256) {
    const int b = it % nc, kg = it / nc;
    int l = (int)sqrtf((float)b);
    l += (l + 1) * (l + 1) <= b;
    l -= l * l > b;
    const int m = b - l * l - l;
    // D[m][q] read as (-1)^(m+q) D[q][m], along the lanes
    const int odd = m < 0, am = odd ? -m : m, dd = odd ? l : l + 1, sg = odd ? -1 : 1;
    const double* D = dw + rot_offset(l) + (odd ? (l + 1) * (l + 1) + am - 1 : am);
    const double* c = C1 + 4 * kg * nc + l * l + l;
    double v[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int q = odd; q <= l; ++q, D += dd) {
      const double d = (am + q) & 1 ? -*D : *D;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = fma(d, c[k * nc + sg * q], v[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) C2[(4 * kg + k) * nc + b] = v[k];
  }
  __syncthreads();
  // colatitude sums of F: e[k][j][m] over C1's place and beyond, C2 moved to the front first
  for (int it = tid; it < 12 * nc; it += 256) C1[it] = C2[it];
  __syncthreads();
  const int nm = 2 * p + 1;
  double* ev = work + 12 * nc;  // [12][p1][nm]
  for (int it = tid; it < p1 * nm; it += 256) {
    const int j = it / nm, m = it % nm - p, am = m < 0 ? -m : m;
    const double* G = tab + T.gg + (size_t)j * nc + m;
    const double* c = C1 + m;
    double v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = 0.0;
#pragma unroll 4
    for (int l = am; l <= p; ++l) {
      const double g = G[l * l + l];
#pragma unroll
      for (int k = 0; k < 12; ++k) v[k] = fma(g, c[k * nc + l * l + l], v[k]);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) ev[k * p1 * nm + it] = v[k];
  }
  __syncthreads();
  const int ci[6] = {0, 1, 2, 0, 0, 1}, cj[6] = {0, 1, 2, 1, 2, 2};
  double* S = Sop + (size_t)s * M3 * M3;
  double* K = Kop + (size_t)s * M3 * M3;
  // azimuths sh and -sh from the target's together: their cosine parts agree, the sine parts
  // differ in sign
  for (int it = tid; it < p1 * p1; it += 256) {
    const int j = it / p1, sh = it % p1;
    const double* q = ev + j * nm + p;
    double ve[12], vo[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      ve[k] = q[k * p1 * nm];
      vo[k] = 0.0;
    }
    int r = 0;
    for (int m = 1; m <= p; ++m) {
      r += sh;
      r -= r >= 2 * p ? 2 * p : 0;
      const double cm = az[r], sm = az[2 * p + r];
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        ve[k] = fma(q[k * p1 * nm + m], cm, ve[k]);
        vo[k] = fma(q[k * p1 * nm - m], sm, vo[k]);
      }
    }
    for (int g = 0; g < (sh == 0 || sh == p ? 1 : 2); ++g) {
      int ka = g ? kt - sh : kt + sh;
      ka += ka < 0 ? 2 * p : 0;
      ka -= ka >= 2 * p ? 2 * p : 0;
      const int a = j * 2 * p + ka;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int c = ci[k], cc = cj[k];
        const double vs = g ? ve[k] - vo[k] : ve[k] + vo[k], vk = g ? ve[6 + k] - vo[6 + k] : ve[6 + k] + vo[6 + k];
        const size_t at = (size_t)(c * M + t) * M3 + cc * M + a;
        S[at] = vs;
        K[at] = vk;
        if (c != cc) {
          const size_t bt = (size_t)(cc * M + t) * M3 + c * M + a;
          S[bt] = vs;
          K[bt] = vk;
        }
      }
    }
  }
}

hipError_t launch_singular_assemble(int ns, int p, int ps, double eta, const double* coef, const double* gn,
                                    const double* glr_t, const double* glt, const double* glw,
                                    const double* rW, double* tab, double* Sop, double* Kop, hipStream_t st) {
  const SingularTables T = singular_tables(p, ps);
  k_singular_tables<<<T.NIP * T.MP / 64 + 1, 64, 0, st>>>(T, glr_t, glt, glw, tab);
  k_rotation_matrices<<<dim3(((p + 1) * (p + 1) + 63) / 64, p + 1), 64, 0, st>>>(p, glt, tab + T.dw);
  const int nc = (p + 1) * (p + 1), MQ = (p + 1 + 3) / 4 * 4;
  const size_t lds = (size_t)(6 * MQ * (p + 1) + 4 * p + singular_work(p)) * sizeof(double);
  const dim3 grid((p + 1) * 2 * p, ns);
  auto run = [&](auto kern) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kern<<<grid, 256, lds, st>>>(T, eta, coef, gn, rW, tab, Sop, Kop);
    return hipGetLastError();
  };
  // (l, m) x 3 sums per thread: 507 at p = 12, 768 at p = 15, 1323 at p = 20
  if (3 * nc <= 512) return run(k_singular<2, 1>);
  if (p <= 15) return run(k_singular<3, 1>);
  return run(k_singular<6, 2>);
}

}  // namespace rbm
