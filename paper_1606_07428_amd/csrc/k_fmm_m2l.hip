// Multipole-to-local translations of the fast multipole far field (k_fmm.hip) in float32, orders
// up to 15, on the matrix cores: every displacement a = c_t - c_s = v w is rotated onto the z axis,
//   M'' = T1(v) M,   L''_k = sum_n h_{n+k} M''_n per order m,   L += T2(v) L'',
// with h_j = j! / |a|^(j+1) and T1, T2 block diagonal in the degree.  With D_n of the rotation by the
// polar angle of v (real, cosines and sines) and phi its azimuth,
//   T1: Re, Im of M_n^m -> c_n^m = Re M''_n^m and s_n^m = -Im M''_n^m,
//   T2: c, s of L'' -> Re, Im of L_k^l, with the sign (-1)^(k + m) of the translation.
// The factors that turn the factorial normalisation into the orthonormal one, in which D_n is
// orthogonal, are folded into T1 and T2.  The tables depend on v and the order alone.
//
// About 2 (2/3 p^3) + p^3/3 multiply-adds a displacement and density instead of the p^4 of the
// dense translation (5.1 thousand instead of 29 thousand at p = 12), and the rotations are
// products for the matrix cores: a wave takes four target boxes of one octant (the same child of
// their parents, so all have the same displacements) times four densities as the 16 columns of
// v_mfma_f32_16x16x4.  Rows of a tile: cosine (Re) and sine (Im) of 8 orders, row 2 m + part; orders
// 8.. of degrees 8.. make a second tile.  A product's output rows 4 g + e lie where the next one,
// taken in k-steps e, wants its input rows, so the state stays in registers throughout; the
// translation along z couples the degrees of one row, register by register.  A lane's rows are two
// whole coefficients of one density, so it loads and stores them in complex numbers.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "fmm.h"
#include "kernels.h"

namespace rbm {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

// k-steps of a degree's tiles: input rows 4 g + e of the first tile are orders 2 g, 2 g + 1, of the
// second orders 8 more.  A group of four steps per (out tile, in tile), one float4 per lane, in the
// order (U, U), (U, V), (V, U), (V, V); degree 0 needs its first step alone, degree 8 two of in tile V.
__host__ __device__ constexpr int ksteps_u(int n) { return n > 0 ? 4 : 1; }
__host__ __device__ constexpr int ksteps_v(int n) { return n > 8 ? 4 : 2; }
__host__ __device__ constexpr int groups_of(int n) { return n < 8 ? 1 : 4; }
__host__ __device__ constexpr int group0(int n) { return n < 8 ? n : 8 + 4 * (n - 8); }
constexpr int kRotMax = kFmmRotOrder;
constexpr int kRotGroups = group0(kRotMax + 1);
constexpr size_t kRotFloats = (size_t)kRotGroups * 256;
constexpr int kRotVecs = 343;
constexpr int kRotH = 2 * kRotMax + 2;

// tables: T1, T2 of every v, then h of every level and v, then a box of zeros
static size_t rot_h_at() { return 2 * kRotVecs * kRotFloats; }
static size_t rot_zero_at(int levels) { return rot_h_at() + (size_t)levels * kRotVecs * kRotH; }
size_t fmm_rotation_floats(int max_level) {
  return rot_zero_at(max_level - 1) + 8 * (kRotMax + 1) * (kRotMax + 2) / 2;
}

__global__ void k_fmm_rot_zero(size_t n4, f4* __restrict__ tab) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) tab[i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
}

// d^l_{M,M'} by its recurrence in l, from l = max(M, |M'|); c = cos(theta/2), s = sin(theta/2); M >= 0.
struct WignerStep {
  int l, M, Mp;
  double ct, q0, v, prev;
  __device__ __forceinline__ WignerStep(int M_, int Mp_, double ct_, double c, double s) : M(M_), Mp(Mp_), ct(ct_) {
    l = max(M, abs(Mp));
    const int ec = abs(M + Mp), es = abs(M - Mp);
    double binom = 1.0;
    for (int k = 1; k <= ec; ++k) binom = binom * (2 * l - ec + k) / k;
    v = sqrt(binom);
    for (int k = 0; k < ec; ++k) v *= c;
    for (int k = 0; k < es; ++k) v *= s;
    if (Mp > M && (es & 1)) v = -v;
    prev = q0 = 0.0;
  }
  __device__ __forceinline__ void step() {
    const double l1 = l + 1.0, q1 = (l1 * l1 - (double)(M * M)) * (l1 * l1 - (double)(Mp * Mp));
    const double next =
        l == 0 ? ct * v : ((2.0 * l + 1.0) * (l * l1 * ct - M * Mp) * v - l1 * sqrt(q0) * prev) / (l * sqrt(q1));
    prev = v;
    v = next;
    q0 = q1;
    ++l;
  }
};

// Place of entry (out row, in row) of degree n, row 2 m + part within tile m >> 3.
__device__ __forceinline__ void rot_put(float* T, int n, int mo, int po, int mi, int pi, double v) {
  const int ri = 2 * (mi & 7) + pi, lane = (ri >> 2) * 16 + 2 * (mo & 7) + po;
  const int group = group0(n) + 2 * (mo >> 3) + (mi >> 3);
  T[((size_t)group * 64 + lane) * 4 + (ri & 3)] = (float)v;
}

// T1 and T2, a thread per (v, m, m'); h, a thread per (level, v).
__global__ __launch_bounds__(64) void k_fmm_rot_tables(int P, int L, double D, float* __restrict__ tab, size_t h_at) {
  const int v = blockIdx.x, vx = v % 7 - 3, vy = (v / 7) % 7 - 3, vz = v / 49 - 3;
  if (abs(vx) <= 1 && abs(vy) <= 1 && abs(vz) <= 1) return;
  const double r = sqrt((double)(vx * vx + vy * vy + vz * vz)), ct = vz / r;
  if (blockIdx.y == gridDim.y - 1) {
    const int lev = 2 + threadIdx.x;
    if (lev > L) return;
    float* h = tab + h_at + ((size_t)(lev - 2) * kRotVecs + v) * kRotH;
    const double ir = 1.0 / (r * ldexp(D, -lev));
    double x = ir;
    for (int j = 0; j < kRotH; ++j) {
      h[j] = j <= 2 * P ? (float)x : 0.0f;
      x *= (j + 1) * ir;
    }
    return;
  }
  const int e = blockIdx.y * 64 + threadIdx.x;
  if (e >= (P + 1) * (P + 1)) return;
  const int m = e / (P + 1), mp = e % (P + 1);
  const double c = sqrt(0.5 * (1.0 + ct)), s = sqrt(0.5 * (1.0 - ct));
  double sm, cm;
  sincos(m * atan2((double)vy, (double)vx), &sm, &cm);
  const double r2 = 1.41421356237309504880;
  const double f0 = (m == 0 ? 1.0 / r2 : 1.0) * (mp == 0 ? 1.0 / r2 : 1.0);
  const double eps = (m ? r2 : 1.0) / (mp ? r2 : 1.0);
  float* T1 = tab + (size_t)(2 * v) * kRotFloats;
  float* T2 = T1 + kRotFloats;
  WignerStep a(m, mp, ct, c, s), b(m, -mp, ct, c, s);
  double q = 1.0;  // (n - m)! (n + m)! / ((n - m')! (n + m')!)
  {
    const int n = a.l, lo = min(m, mp), hi = max(m, mp);
    for (int k = n - hi + 1; k <= n - lo; ++k) q *= k;
    for (int k = n + lo + 1; k <= n + hi; ++k) q /= k;
    if (m > mp) q = 1.0 / q;
  }
  for (int n = a.l;; ++n) {
    const double sb = mp & 1 ? -b.v : b.v;
    const double dc = f0 * (a.v + sb), ds = m > 0 && mp > 0 ? a.v - sb : 0.0;
    const double w = sqrt(q), w1 = w * eps, w2 = (n + mp) & 1 ? -w / eps : w / eps;
    rot_put(T1, n, mp, 0, m, 0, dc * cm * w1);
    rot_put(T1, n, mp, 0, m, 1, -dc * sm * w1);
    rot_put(T1, n, mp, 1, m, 0, -ds * sm * w1);
    rot_put(T1, n, mp, 1, m, 1, -ds * cm * w1);
    rot_put(T2, n, m, 0, mp, 0, dc * cm * w2);
    rot_put(T2, n, m, 0, mp, 1, -ds * sm * w2);
    rot_put(T2, n, m, 1, mp, 0, dc * sm * w2);
    rot_put(T2, n, m, 1, mp, 1, ds * cm * w2);
    if (n == P) break;
    q *= (n + 1.0 - m) * (n + 1.0 + m) / ((n + 1.0 - mp) * (n + 1.0 + mp));
    a.step();
    b.step();
  }
}

// f(std::integral_constant<int, I>) for I = B .. E - 1
template <int B, int E, class F>
__host__ __device__ __forceinline__ void each(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    each<B + 1, E>(f);
  }
}

template <int CTRL>
__device__ __forceinline__ float quad(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Bound: the 57 KB of tables that a wave reads per displacement (10 GB in all at p = 12 and 4096 leaves,
// 7.8 TB/s from L2) and the latency of two waves per SIMD; matrix cores 34% busy, vector units about
// as much.  Operands are loaded two degrees ahead (256 registers at order 12, 6 spilled).  5.1 (dense, on the
// vector units) -> 1.45 ms.  The
// whole sum's rounding error against float64 on the same tree falls from 2.4e-6 to 2.0e-6 (rms).
// Workgroup: 4 boxes of one octant of a level; its NW waves take every NWth displacement and add their
// locals through LDS.  (Eight waves: two per SIMD, and enough workgroups to even out over the CUs.)
template <int P, int NW>
__global__ __launch_bounds__(64 * NW) void k_fmm_m2l_rot(int L, double D, FmmLevels lv,
                                                         const float* __restrict__ tab, size_t h_at,
                                                         const float* __restrict__ zero,
                                                         const Cx<float>* __restrict__ Mexp,
                                                         Cx<float>* __restrict__ Lexp) {
  constexpr int NV = P < 8 ? 0 : P - 7, NR = P + 1 + NV;
  extern __shared__ f4 part[];  // [NW / 2][NR][64]
  int lev = L;  // the last level first: it has the longest lists
  while (lev > 2 && (int)blockIdx.x >= lv.first[lev - 1]) --lev;
  const int wg = (int)blockIdx.x - lv.first[lev], nl = 1 << lev, hl = nl / 2;
  const int per = hl * hl * hl / 4, oct = wg / per;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g = lane >> 4, dens = col & 3;
  const int ox = oct & 1, oy = (oct >> 1) & 1, oz = oct >> 2;
  const int* cnt = lv.cnt[lev];
  struct Box {
    int i, j, k;
  };
  auto box = [&](int n) {  // the workgroup's box n
    const int q = (wg % per) * 4 + n;
    return Box{2 * (q % hl) + ox, 2 * ((q / hl) % hl) + oy, 2 * (q / (hl * hl)) + oz};
  };
  auto place = [&](int i, int j, int k) { return (k * nl + j) * nl + i; };
  const Box home = box(col >> 2);
  const int b = place(home.i, home.j, home.k);
  if (!__any(cnt[b] > 0)) return;  // the same boxes in every wave
  // Displacements with points at both ends, all looked up at once: bit r of `some` for box lane & 3 and this
  // wave's displacement 16 r + lane / 4.  The others are not computed: in a cube of bodies they are few, in a
  // sheet or a chain most (order 12, float32, whole sum: 3000 points in a chain 1061 -> 660 us, 6000 along a
  // diagonal 2084 -> 1060; the translations of a sheet of 200,000 709 -> 134).
  constexpr int kPer = 216 / NW;
  static_assert(216 % NW == 0 && kPer <= 64, "displacements of a wave");
  unsigned some = 0;
  {
    const Box s = box(lane & 3);
    const bool here = cnt[place(s.i, s.j, s.k)] > 0;
#pragma unroll
    for (int r = 0; r < (kPer + 15) / 16; ++r) {
      const int k = 16 * r + (lane >> 2), d = wv + NW * k;
      const int vx = d % 6 - 3 + ox, vy = (d / 6) % 6 - 3 + oy, vz = d / 36 - 3 + oz;
      const int si = s.i - vx, sj = s.j - vy, sk = s.k - vz;
      const bool far = abs(vx) > 1 || abs(vy) > 1 || abs(vz) > 1;
      if (here && k < kPer && far && (unsigned)si < (unsigned)nl && (unsigned)sj < (unsigned)nl &&
          (unsigned)sk < (unsigned)nl && cnt[place(si, sj, sk)] > 0)
        some |= 1u << r;
    }
  }
  const int Kc = tri(P + 1, 0);
  const f2* Mlev = reinterpret_cast<const f2*>(Mexp + lv.off[lev] * 4 * Kc) + dens;
  const f2* zl = reinterpret_cast<const f2*>(zero) + dens;
  const float w = (float)ldexp(D, -lev);
  const float psi = dens == 3 ? -w : 0.0f;
  f4 accU[P + 1], accV[NV + 1], U[P + 1], V[NV + 1];
#pragma unroll
  for (int n = 0; n <= P; ++n) accU[n] = U[n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int n = 0; n <= NV; ++n) accV[n] = V[n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int it = 0; it < kPer; ++it) {
    const unsigned boxes = (unsigned)(__ballot(some >> (it >> 4) & 1) >> 4 * (it & 15)) & 15;
    if (boxes == 0) continue;
    const int d = wv + NW * it, vx = d % 6 - 3 + ox, vy = (d / 6) % 6 - 3 + oy, vz = d / 36 - 3 + oz;
    const int v = ((vz + 3) * 7 + (vy + 3)) * 7 + (vx + 3);
    const f2* src = boxes >> (col >> 2) & 1 ? Mlev + (size_t)(b - place(vx, vy, vz)) * 4 * Kc : zl;
    const f4* T1 = reinterpret_cast<const f4*>(tab + (size_t)(2 * v) * kRotFloats) + lane;
    const f4* T2 = T1 + kRotFloats / 4;
    const float* h = tab + h_at + ((size_t)(lev - 2) * kRotVecs + v) * kRotH;
    const float ax = psi * vx, ay = psi * vy, az = psi * vz;
    // coefficients (n, 8 t + 2 g), (n, 8 t + 2 g + 1) of this lane's box and density; the psi expansion
    // about the target's centre: psi - a . phi.  Orders above n meet zeros of T1.
    auto shift = [&](f4 v) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = fmaf(ax, quad<0x00>(v[e]), fmaf(ay, quad<0x55>(v[e]), fmaf(az, quad<0xAA>(v[e]), v[e])));
      return v;
    };
    auto load = [&](int n, int t) {
      const f2 a = src[4 * (tri(n, 0) + min(8 * t + 2 * g, n))], b = src[4 * (tri(n, 0) + min(8 * t + 2 * g + 1, n))];
      return f4{a.x, a.y, b.x, b.y};
    };
    // operands of a degree, loaded kAhead degrees before they are used
    constexpr int kAhead = 2;
    f4 x[kAhead + 1], z[kAhead + 1], ta[kAhead + 1][4];
    auto fetch = [&](auto in, const f4* T, bool data) {
      constexpr int n = in, at = n % (kAhead + 1);
      if constexpr (n <= P) {
        if (data) {
          x[at] = load(n, 0);
          if constexpr (n >= 8) z[at] = load(n, 1);
        }
        each<0, groups_of(n)>([&](auto k) { ta[at][k] = T[(group0(n) + k) * 64]; });
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](f4 t, f4 v, auto steps, f4& y) {
      each<0, decltype(steps)::value>([&](auto e) {
        y = __builtin_amdgcn_mfma_f32_16x16x4f32(t[(int)e], v[(int)e], y, 0, 0, 0);
      });
    };
    each<0, kAhead>([&](auto in) { fetch(in, T1, true); });
    each<0, P + 1>([&](auto in) {
      constexpr int n = in, at = n % (kAhead + 1), nv = n < 8 ? 0 : n - 8;
      fetch(std::integral_constant<int, n + kAhead>{}, T1, true);
      const std::integral_constant<int, ksteps_u(n)> ku;
      const std::integral_constant<int, ksteps_v(n)> kv;
      const f4 xs = shift(x[at]);
      f4 u{0.0f, 0.0f, 0.0f, 0.0f};
      mul(ta[at][0], xs, ku, u);
      if constexpr (n >= 8) {
        const f4 zs = shift(z[at]);
        f4 t{0.0f, 0.0f, 0.0f, 0.0f};
        mul(ta[at][2], xs, ku, t);
        mul(ta[at][1], zs, kv, u);
        mul(ta[at][3], zs, kv, t);
        V[nv] = t;
      }
      U[n] = u;
    });
    each<0, kAhead>([&](auto in) { fetch(in, T2, false); });
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float t[P + 1];
#pragma unroll
      for (int k = 0; k <= P; ++k) {
        t[k] = 0.0f;
#pragma unroll
        for (int n = 0; n <= P; ++n) t[k] = fmaf(h[n + k], U[n][e], t[k]);
      }
#pragma unroll
      for (int k = 0; k <= P; ++k) U[k][e] = t[k];
#pragma unroll
      for (int k = 8; k <= P; ++k) {
        t[k] = 0.0f;
#pragma unroll
        for (int n = 8; n <= P; ++n) t[k] = fmaf(h[n + k], V[n - 8][e], t[k]);
      }
#pragma unroll
      for (int k = 8; k <= P; ++k) V[k - 8][e] = t[k];
    }
    each<0, P + 1>([&](auto in) {
      constexpr int n = in, at = n % (kAhead + 1), nv = n < 8 ? 0 : n - 8;
      fetch(std::integral_constant<int, n + kAhead>{}, T2, false);
      const std::integral_constant<int, ksteps_u(n)> ku;
      const std::integral_constant<int, ksteps_v(n)> kv;
      mul(ta[at][0], U[n], ku, accU[n]);
      if constexpr (n >= 8) {
        mul(ta[at][2], U[n], ku, accV[nv]);
        mul(ta[at][1], V[nv], kv, accU[n]);
        mul(ta[at][3], V[nv], kv, accV[nv]);
      }
    });
  }
#pragma unroll
  for (int half = NW / 2; half > 0; half /= 2) {
    f4* mine = part + (size_t)(wv % half) * NR * 64 + lane;
    if (wv >= half && wv < 2 * half) {
#pragma unroll
      for (int n = 0; n <= P; ++n) mine[n * 64] = accU[n];
#pragma unroll
      for (int n = 0; n < NV; ++n) mine[(P + 1 + n) * 64] = accV[n];
    }
    __syncthreads();
    if (wv < half) {
#pragma unroll
      for (int n = 0; n <= P; ++n) accU[n] += mine[n * 64];
#pragma unroll
      for (int n = 0; n < NV; ++n) accV[n] += mine[(P + 1 + n) * 64];
    }
    __syncthreads();
  }
  if (wv > 0 || cnt[b] == 0) return;
  f2* out = reinterpret_cast<f2*>(Lexp + (lv.off[lev] + (size_t)b) * 4 * Kc) + dens;
  each<0, P + 1>([&](auto in) {
    constexpr int n = in, nv = n < 8 ? 0 : n - 8;
    auto put = [&](int m, f4 v) {
      if (m <= n) out[4 * (tri(n, 0) + m)] = f2{v.x, v.y};
      if (m + 1 <= n) out[4 * (tri(n, 0) + m + 1)] = f2{v.z, v.w};
    };
    put(2 * g, accU[n]);
    if (n >= 8) put(8 + 2 * g, accV[nv]);
  });
}

hipError_t launch_fmm_rotations(int P, int L, int max_level, double D, float* tab, hipStream_t st) {
  if (P < 2 || P > kRotMax || L < 2 || L > max_level) return hipErrorInvalidValue;
  const size_t n4 = fmm_rotation_floats(max_level) / 4;
  k_fmm_rot_zero<<<(n4 + 255) / 256, 256, 0, st>>>(n4, reinterpret_cast<f4*>(tab));
  k_fmm_rot_tables<<<dim3(kRotVecs, ((P + 1) * (P + 1) + 63) / 64 + 1), 64, 0, st>>>(P, L, D, tab, rot_h_at());
  return hipGetLastError();
}

hipError_t launch_fmm_m2l_rot(int P, int L, int max_level, double D, FmmLevels lv, const float* tab,
                              const Cx<float>* Mexp, Cx<float>* Lexp, hipStream_t st) {
  if (P < 2 || P > kRotMax || L < 2 || L > 6) return hipErrorInvalidValue;
  int nwg = 0;
  for (int lev = L; lev >= 2; --lev) {
    lv.first[lev] = nwg;
    nwg += 1 << (3 * lev - 2);
  }
  const float* zero = tab + rot_zero_at(max_level - 1);
  auto run = [&](auto order) {
    constexpr int n = decltype(order)::value, nr = n < 8 ? n + 1 : 2 * n - 6;
    constexpr int nw = n <= 12 ? 8 : 4;  // above 12 the state takes more than half of the registers
    const auto kern = k_fmm_m2l_rot<n, nw>;
    const int lds = nw / 2 * nr * 64 * (int)sizeof(f4);
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<nwg, 64 * nw, lds, st>>>(L, D, lv, tab, rot_h_at(), zero, Mexp, Lexp);
    return hipGetLastError();
  };
  hipError_t e = hipErrorInvalidValue;
  each<2, kRotMax + 1>([&](auto order) {
    if (P == order) e = run(order);
  });
  return e;
}

}  // namespace rbm
