// Setup kernels (float64): grid tables, shape geometry, A0 and the velocity functional.  §2.2, §2.3, §3, §3.1, §3.2 of the paper.
#include "common.h"
#include "kernels.h"

namespace rbm {

// n-point Gauss-Legendre nodes (ascending) and weights by Newton's method on P_n.
__global__ void k_gauss_legendre(int n, double* t, double* w) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double x = -cos(RBM_PI * (i + 0.75) / (n + 0.5));
  double pn = 0.0, pn1 = 0.0;
  for (int it = 0; it < 100; ++it) {
    double p0 = 1.0, p1 = x;
    for (int k = 2; k <= n; ++k) {
      const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    pn = p1;
    pn1 = p0;
    const double dp = n * (x * pn - pn1) / (x * x - 1.0);
    const double dx = pn / dp;
    x -= dx;
    if (fabs(dx) < 1e-16) break;
  }
  double p0 = 1.0, p1 = x;
  for (int k = 2; k <= n; ++k) {
    const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
    p0 = p1;
    p1 = p2;
  }
  const double dp = n * (x * p1 - p0) / (x * x - 1.0);
  t[i] = x;
  w[i] = 2.0 / ((1.0 - x * x) * dp * dp);
}

hipError_t launch_gauss_legendre(int n, double* t, double* w, hipStream_t st) {
  k_gauss_legendre<<<(n + 63) / 64, 64, 0, st>>>(n, t, w);
  return hipGetLastError();
}

// Per grid node a: real SH tables and the forward transform (§3 grid, band B_p).
__global__ void k_grid_tables(int p, const double* glt, const double* glw, double* Y, double* Yt,
                              double* Yps, double* F, double* Ft, double* nth, double* nph,
                              double* nlam) {
  const int M = (p + 1) * 2 * p;
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= M) return;
  const int nB = p * p + 2 * p;
  const int j = a / (2 * p), k = a % (2 * p);
  const double x = glt[j];
  const double s = sqrt(fmax(0.0, 1.0 - x * x));
  const double ph = RBM_PI * k / p;
  const double lam = glw[j];
  nth[a] = acos(x);
  nph[a] = ph;
  nlam[a] = lam;
  const double wq = RBM_PI / p * lam;
  int cur_m = -1;
  double cm = 1.0, sm = 0.0;
  legendre_sweep(p, x, s, [&](int l, int m, double P, double Q, double D) {
    const int i0 = l * l + l;
    if (m == 0) {
      Y[(size_t)i0 * M + a] = P;
      Yt[(size_t)i0 * M + a] = D;
      Yps[(size_t)i0 * M + a] = 0.0;
      const int b = band_index(l, 0, p);
      F[(size_t)b * M + a] = wq * P;
      Ft[(size_t)a * nB + b] = wq * P;
      return;
    }
    if (m != cur_m) {
      sincos(m * ph, &sm, &cm);
      cur_m = m;
    }
    const double r2 = 1.41421356237309504880;
    const double yp = r2 * P * cm, ym = r2 * P * sm;
    Y[(size_t)(i0 + m) * M + a] = yp;
    Y[(size_t)(i0 - m) * M + a] = ym;
    Yt[(size_t)(i0 + m) * M + a] = r2 * D * cm;
    Yt[(size_t)(i0 - m) * M + a] = r2 * D * sm;
    Yps[(size_t)(i0 + m) * M + a] = -r2 * m * Q * sm;
    Yps[(size_t)(i0 - m) * M + a] = r2 * m * Q * cm;
    const int bp = band_index(l, m, p);
    const double nu = (l == p && m == p) ? 0.5 : 1.0;
    F[(size_t)bp * M + a] = wq * nu * yp;
    Ft[(size_t)a * nB + bp] = wq * nu * yp;
    const int bm = band_index(l, -m, p);
    if (bm >= 0) {
      F[(size_t)bm * M + a] = wq * ym;
      Ft[(size_t)a * nB + bm] = wq * ym;
    }
  });
}

hipError_t launch_grid_tables(int p, const double* gl_t, const double* gl_w, double* Ytab,
                              double* Yttab, double* Ypstab, double* Ftab, double* Fttab,
                              double* node_th, double* node_ph, double* node_lam, hipStream_t st) {
  const int M = (p + 1) * 2 * p;
  k_grid_tables<<<(M + 63) / 64, 64, 0, st>>>(p, gl_t, gl_w, Ytab, Yttab, Ypstab, Ftab, Fttab,
                                              node_th, node_ph, node_lam);
  return hipGetLastError();
}

// Rotated GL(ps+1) x trapezoid(2ps) grid and the singular weights
// W_jk = (pi/ps) lam'_j [sum_{nu<=ps} P_nu(t'_j)] sqrt(2(1-t'_j)): since
// 1/|e_z - s'| = sum_nu P_nu(t'), this integrates circle averages of degree <= ps
// in t' exactly against the 1/r singularity at the rotated pole.
__global__ void k_rotated_rule(int ps, const double* glt, const double* glw, double* nodes,
                               double* W) {
  const int Ms = (ps + 1) * 2 * ps;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Ms) return;
  const int j = q / (2 * ps), k = q % (2 * ps);
  const double t = glt[j];
  double pm1 = 0.0, p0 = 1.0, S = 1.0;
  for (int nu = 1; nu <= ps; ++nu) {
    const double pn = ((2.0 * nu - 1.0) * t * p0 - (nu - 1.0) * pm1) / nu;
    pm1 = p0;
    p0 = pn;
    S += pn;
  }
  const double ph = RBM_PI * k / ps;
  const double st = sqrt(fmax(0.0, 1.0 - t * t));
  double sp, cp;
  sincos(ph, &sp, &cp);
  nodes[q] = st * cp;
  nodes[Ms + q] = st * sp;
  nodes[2 * Ms + q] = t;
  W[q] = RBM_PI / ps * glw[j] * S * sqrt(2.0 * (1.0 - t));
}

hipError_t launch_rotated_rule(int ps, const double* glt, const double* glw, double* nodes,
                               double* W, hipStream_t st) {
  const int Ms = (ps + 1) * 2 * ps;
  k_rotated_rule<<<(Ms + 63) / 64, 64, 0, st>>>(ps, glt, glw, nodes, W);
  return hipGetLastError();
}

// Radial shape r(s) = sum rc Y -> coordinate coefficients of x = r(s) s by the
// exact forward transform of the grid values (degree of x below p).
__global__ __launch_bounds__(256) void k_radial_to_coef(int p, int nrc, const double* rc_all,
                                                        const double* Ytab, const double* Ftab,
                                                        const double* nth, const double* nph,
                                                        double* coef_all) {
  extern __shared__ double xg[];  // [3][M]
  const int M = (p + 1) * 2 * p, nc = (p + 1) * (p + 1), nB = p * p + 2 * p;
  const int s = blockIdx.x;
  const double* rc = rc_all + (size_t)s * nrc;
  for (int a = threadIdx.x; a < M; a += blockDim.x) {
    double r = 0.0;
    for (int i = 0; i < nrc; ++i) r += rc[i] * Ytab[(size_t)i * M + a];
    double st, ct, sp, cp;
    sincos(nth[a], &st, &ct);
    sincos(nph[a], &sp, &cp);
    xg[a] = r * st * cp;
    xg[M + a] = r * st * sp;
    xg[2 * M + a] = r * ct;
  }
  __syncthreads();
  double* coef = coef_all + (size_t)s * 3 * nc;
  for (int b = threadIdx.x; b < nB; b += blockDim.x) {
    const int full = b < p * p ? b : b + 1;
    for (int c = 0; c < 3; ++c) {
      double v = 0.0;
      for (int a = 0; a < M; ++a) v += Ftab[(size_t)b * M + a] * xg[c * M + a];
      coef[c * nc + full] = v;
    }
  }
  if (threadIdx.x < 3) coef[threadIdx.x * nc + p * p] = 0.0;  // the dropped (p, -p) mode
}

hipError_t launch_radial_to_coef(int ns, int p, int nrc, const double* rc, const double* Ytab,
                                 const double* Ftab, const double* node_th, const double* node_ph,
                                 double* coef, hipStream_t st) {
  const int M = (p + 1) * 2 * p;
  k_radial_to_coef<<<ns, 256, 3 * M * sizeof(double), st>>>(p, nrc, rc, Ytab, Ftab, node_th,
                                                            node_ph, coef);
  return hipGetLastError();
}

// Per shape: x, outward normal, J = |x_theta x x_phi/sin|, weights w = (pi/p) lam J (§3),
// area, area centroid, tau (§2.2) and tau^{-1}; r = x - x^c.
// shp layout per shape (32 doubles): [0] area, [1..3] xc, [4..12] tau, [13..21] tau^{-1}.
__global__ __launch_bounds__(256) void k_shape_geometry(int p, const double* coef_all,
                                                        const double* Ytab, const double* Yttab,
                                                        const double* Ypstab, const double* nlam,
                                                        double* gx_all, double* gn_all,
                                                        double* gw_all, double* gr_all,
                                                        double* shp_all) {
  __shared__ double red[16];
  const int M = (p + 1) * 2 * p, nc = (p + 1) * (p + 1);
  const int s = blockIdx.x;
  const double* coef = coef_all + (size_t)s * 3 * nc;
  double* gx = gx_all + (size_t)s * 3 * M;
  double* gn = gn_all + (size_t)s * 3 * M;
  double* gw = gw_all + (size_t)s * M;
  double* gr = gr_all + (size_t)s * 3 * M;
  double a_area = 0.0, a_x[3] = {0.0, 0.0, 0.0};
  for (int a = threadIdx.x; a < M; a += blockDim.x) {
    double x[3] = {0, 0, 0}, xt[3] = {0, 0, 0}, xp[3] = {0, 0, 0};
    for (int i = 0; i < nc; ++i) {
      const double y = Ytab[(size_t)i * M + a], yt = Yttab[(size_t)i * M + a],
                   yp = Ypstab[(size_t)i * M + a];
      for (int c = 0; c < 3; ++c) {
        const double cf = coef[c * nc + i];
        x[c] += cf * y;
        xt[c] += cf * yt;
        xp[c] += cf * yp;
      }
    }
    const double cx = xt[1] * xp[2] - xt[2] * xp[1];
    const double cy = xt[2] * xp[0] - xt[0] * xp[2];
    const double cz = xt[0] * xp[1] - xt[1] * xp[0];
    const double J = sqrt(cx * cx + cy * cy + cz * cz);
    const double w = RBM_PI / p * nlam[a] * J;
    for (int c = 0; c < 3; ++c) gx[c * M + a] = x[c];
    gn[a] = cx / J;
    gn[M + a] = cy / J;
    gn[2 * M + a] = cz / J;
    gw[a] = w;
    a_area += w;
    for (int c = 0; c < 3; ++c) a_x[c] += w * x[c];
  }
  const double area = block_sum(a_area, red);
  double xc[3];
  for (int c = 0; c < 3; ++c) xc[c] = block_sum(a_x[c], red) / area;
  __syncthreads();
  double t6[6] = {0, 0, 0, 0, 0, 0};  // xx, yy, zz (of r r^T), xy, xz, yz; and |r|^2 via sum
  for (int a = threadIdx.x; a < M; a += blockDim.x) {
    double r[3];
    for (int c = 0; c < 3; ++c) {
      r[c] = gx[c * M + a] - xc[c];
      gr[c * M + a] = r[c];
    }
    const double w = gw[a];
    t6[0] += w * r[0] * r[0];
    t6[1] += w * r[1] * r[1];
    t6[2] += w * r[2] * r[2];
    t6[3] += w * r[0] * r[1];
    t6[4] += w * r[0] * r[2];
    t6[5] += w * r[1] * r[2];
  }
  double T[6];
  for (int k = 0; k < 6; ++k) T[k] = block_sum(t6[k], red);
  if (threadIdx.x == 0) {
    double* sp = shp_all + (size_t)s * 32;
    const double tr = T[0] + T[1] + T[2];
    double tau[9] = {tr - T[0], -T[3], -T[4], -T[3], tr - T[1], -T[5], -T[4], -T[5], tr - T[2]};
    sp[0] = area;
    sp[1] = xc[0];
    sp[2] = xc[1];
    sp[3] = xc[2];
    for (int k = 0; k < 9; ++k) sp[4 + k] = tau[k];
    inv3(tau, sp + 13);
  }
}

hipError_t launch_shape_geometry(int ns, int p, const double* coef, const double* Ytab,
                                 const double* Yttab, const double* Ypstab, const double* node_lam,
                                 double* gx, double* gn, double* gw, double* gr, double* shp,
                                 hipStream_t st) {
  k_shape_geometry<<<ns, 256, 0, st>>>(p, coef, Ytab, Yttab, Ypstab, node_lam, gx, gn, gw, gr, shp);
  return hipGetLastError();
}

// A0 = K^T + 1/2 I + L0, column-major A0 from the row-major singular operator K, with
// L0[(c,a),(c',b)] = w_b [(1 + r_a.r_b) d_cc' - r_b[c] r_a[c']] (the augmentation L of §2.3 on
// the grid: int mu + (int r x mu) x r_a).  32 x 32 tiles through LDS, reads and writes along the
// rows of K and the columns of A0.  A0 may not overlap K.
__global__ __launch_bounds__(256) void k_finish_A0(int M, const double* __restrict__ gr_all,
                                                   const double* __restrict__ gw_all,
                                                   const double* __restrict__ K_all, double* __restrict__ A0_all) {
  __shared__ double tile[32][33];
  const int M3 = 3 * M, s = blockIdx.z, r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const double* K = K_all + (size_t)s * M3 * M3;
  const int x = threadIdx.x & 31, y0 = threadIdx.x >> 5;
  for (int y = y0; y < 32; y += 8)
    if (r0 + y < M3 && c0 + x < M3) tile[y][x] = K[(size_t)(r0 + y) * M3 + c0 + x];
  __syncthreads();
  const double* r = gr_all + (size_t)s * 3 * M;
  for (int y = y0; y < 32; y += 8) {
    const int row = r0 + x, col = c0 + y;
    if (row >= M3 || col >= M3) continue;
    const int c = row / M, a = row % M, cc = col / M, b = col % M;
    const double wb = gw_all[(size_t)s * M + b];
    const double ra[3] = {r[a], r[M + a], r[2 * M + a]};
    const double rb[3] = {r[b], r[M + b], r[2 * M + b]};
    const double dot = ra[0] * rb[0] + ra[1] * rb[1] + ra[2] * rb[2];
    double v = wb * ((c == cc ? 1.0 + dot : 0.0) - rb[c] * ra[cc]);
    if (row == col) v += 0.5;
    A0_all[(size_t)s * M3 * M3 + (size_t)col * M3 + row] = tile[x][y] + v;
  }
}

hipError_t launch_finish_A0(int ns, int M, const double* gr, const double* gw, const double* K, double* A0,
                            hipStream_t st) {
  const int n = (3 * M + 31) / 32;
  k_finish_A0<<<dim3(n, n, ns), 256, 0, st>>>(M, gr, gw, K, A0);
  return hipGetLastError();
}

// Velocity functional V0 = G' S0 (6 x 3M per shape, S0 row-major): rows 0..2 average the self
// velocity over the surface, rows 3..5 give tau^{-1} int r x u (§3.3).  64 columns per
// workgroup, each wave a quarter of the nodes, added in wave order.
__global__ __launch_bounds__(256) void k_velocity_functional(int M, const double* __restrict__ Sop,
                                                             const double* __restrict__ gr_all,
                                                             const double* __restrict__ gw_all,
                                                             const double* __restrict__ shp_all,
                                                             double* __restrict__ V0) {
  __shared__ double red[4][6][64];
  const int M3 = 3 * M;
  const int s = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + lane;
  const double* S = Sop + (size_t)s * M3 * M3 + min(col, M3 - 1);
  const double* r = gr_all + (size_t)s * 3 * M;
  const double* w = gw_all + (size_t)s * M;
  const double* sp = shp_all + (size_t)s * 32;
  const double inva = 1.0 / sp[0];
  const double* ti = sp + 13;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int a = wv; a < M; a += 4) {
    const double u0 = S[(size_t)a * M3], u1 = S[(size_t)(M + a) * M3], u2 = S[(size_t)(2 * M + a) * M3];
    const double wa = w[a];
    const double r0 = r[a], r1 = r[M + a], r2 = r[2 * M + a];
    acc[0] += wa * u0 * inva;
    acc[1] += wa * u1 * inva;
    acc[2] += wa * u2 * inva;
    const double x0 = r1 * u2 - r2 * u1, x1 = r2 * u0 - r0 * u2, x2 = r0 * u1 - r1 * u0;
    acc[3] += wa * (ti[0] * x0 + ti[1] * x1 + ti[2] * x2);
    acc[4] += wa * (ti[3] * x0 + ti[4] * x1 + ti[5] * x2);
    acc[5] += wa * (ti[6] * x0 + ti[7] * x1 + ti[8] * x2);
  }
  for (int k = 0; k < 6; ++k) red[wv][k][lane] = acc[k];
  __syncthreads();
  for (int e = threadIdx.x; e < 6 * 64; e += 256) {
    const int k = e / 64, c = e % 64;
    if (blockIdx.x * 64 + c < M3)
      V0[((size_t)s * 6 + k) * M3 + blockIdx.x * 64 + c] = (red[0][k][c] + red[1][k][c]) + (red[2][k][c] + red[3][k][c]);
  }
}

hipError_t launch_velocity_functional(int ns, int M, const double* Sop, const double* gr,
                                      const double* gw, const double* shp, double* V0,
                                      hipStream_t st) {
  k_velocity_functional<<<dim3((3 * M + 63) / 64, ns), 256, 0, st>>>(M, Sop, gr, gw, shp, V0);
  return hipGetLastError();
}

__global__ void k_cast_f32(size_t n, const double* x, float* y) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (float)x[i];
}

__global__ void k_cast_bf16(size_t n, const double* x, uint16_t* y) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float f = (float)x[i];
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (finite inputs)
  y[i] = (uint16_t)(u >> 16);
}

hipError_t launch_cast_f32(size_t n, const double* x, float* y, hipStream_t st) {
  k_cast_f32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, x, y);
  return hipGetLastError();
}

hipError_t launch_cast_bf16(size_t n, const double* x, uint16_t* y, hipStream_t st) {
  k_cast_bf16<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, x, y);
  return hipGetLastError();
}

}  // namespace rbm
