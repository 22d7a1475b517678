// In-place inversion of the shapes' self operators (the block preconditioner of §3.2):
// Gauss-Jordan with partial pivoting, column-major A[j*n + i] = a_ij, float64, blocked by panels
// of kPanel pivots.  Each unblocked step on pivot k: search column k, swap rows k and p,
// scale the pivot row, eliminate column k from every other row, and store the step's
// transformation column in column k.  Within a panel P the steps touch only the panel's
// columns, which then hold the panel's transformation T restricted to P (T differs from I
// only in those columns), so every other column is brought up to date at once: the panel's
// row interchanges, then the rank-kPanel update A(:, J) += (T(:, P) - I_P) A(P, J).  The row
// interchanges are undone at the end as column interchanges.
// Before, one workgroup inverted one matrix with panels of 16 pivots: few shapes left most CUs
// idle, and its updates read the matrix through one CU.  Panels stay one workgroup per matrix
// (the chain of pivot searches); the updates, where the operations are, go over the chip.
// 64 matrices of n = 936: 28.3 -> 9.3 ms (15 panels of 203 us, 15 updates of 373 us, columns
// 0.70 ms); the whole setup of 8 shapes of n = 792: 17.8 -> 6.1 ms, of 35 of n = 1632: 526 -> 339 ms.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace rbm {

constexpr int kPanel = 64;
// ints per matrix behind the n of idx: the panel's row moves (count, then kMoves positions and
// the kMoves positions their contents come from)
constexpr int kMoves = 2 * kPanel;
static_assert(1 + 2 * kMoves <= kInverseInts, "row moves fit the integer scratch");

// (best, row) of the wave in every lane: the largest value, ties to the smallest row.
template <int CTRL>
__device__ __forceinline__ void argmax_dpp(double& best, int& row) {
  const double ov = __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(best), CTRL, 0xf, 0xf, true),
                                     __builtin_amdgcn_mov_dpp(__double2loint(best), CTRL, 0xf, 0xf, true));
  const int oi = __builtin_amdgcn_mov_dpp(row, CTRL, 0xf, 0xf, true);
  if (ov > best || (ov == best && oi < row)) { best = ov; row = oi; }
}
// over each row of 16 lanes
__device__ __forceinline__ void argmax16(double& best, int& row) {
  argmax_dpp<0xB1>(best, row);   // quad_perm [1,0,3,2]
  argmax_dpp<0x4E>(best, row);   // quad_perm [2,3,0,1]
  argmax_dpp<0x141>(best, row);  // row_half_mirror
  argmax_dpp<0x140>(best, row);  // row_mirror
}
__device__ __forceinline__ void argmax_wave(double& best, int& row) {
  argmax16(best, row);
#pragma unroll
  for (int step = 0; step < 2; ++step) {
    auto swap = [&](int v) {
      return step ? __builtin_amdgcn_permlane32_swap(v, v, false, false) : __builtin_amdgcn_permlane16_swap(v, v, false, false);
    };
    const auto lo = swap(__double2loint(best)), hi = swap(__double2hiint(best)), rr = swap(row);
    const double v0 = __hiloint2double((int)hi[0], (int)lo[0]), v1 = __hiloint2double((int)hi[1], (int)lo[1]);
    const int r0 = (int)rr[0], r1 = (int)rr[1];
    const bool second = v1 > v0 || (v1 == v0 && r1 < r0);
    best = second ? v1 : v0;
    row = second ? r1 : r0;
  }
}

// One panel (columns k0 .. k0 + kb) of every matrix, a workgroup each.  A thread owns the rows
// i = tid + 512 r and holds SB of the panel's columns of them in registers; the panel is
// taken in sub-panels of SB columns, each followed by its update of the panel's other columns.
// The pivot's column is always register 0: a step leaves its columns one place lower and
// the column it stores in the last, which keeps the loop over pivots rolled (unrolled, its
// code ran through the instruction cache once per sub-panel: 11 us a pivot).
// idx[k]: the original row now at k.
// Bound: the chain of pivots, two barriers and a search over 512 threads each.
constexpr int kGjThreads = 512;
template <int RP, int SB>
__global__ __launch_bounds__(kGjThreads) void k_gj_panel(int n, int k0, double* __restrict__ A_all,
                                                         int* __restrict__ ints) {
  constexpr int NT = kGjThreads, NW = NT / 64;
  static_assert(NW <= 16 && 2 * SB <= NT, "one row of lanes holds the waves' candidates");
  __shared__ __align__(16) double prow[SB], krow[SB];  // pivot row, row k before the swap
  __shared__ __align__(16) double R[kPanel][SB];       // rows of the sub-panel, other columns
  __shared__ double wval[2][16];
  __shared__ int wrow[2][16];
  __shared__ int pos[NT * RP], spos[NT * RP];        // place of a row in the lists below, or -1
  __shared__ int at[kMoves], from[kMoves], nmove;    // the panel's moves
  __shared__ int sat[2 * SB], sfrom[2 * SB], snmove;  // the sub-panel's
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int s = blockIdx.x, kb = min(kPanel, n - k0);
  double* A = A_all + (size_t)s * n * n;
  int* idx = ints + (size_t)s * (n + kInverseInts);
  int* moves = idx + n;
#pragma unroll
  for (int r = 0; r < RP; ++r) {
    const int i = tid + NT * r;
    if (k0 == 0 && i < n) idx[i] = i;
    pos[i] = i >= k0 && i < k0 + kb ? i - k0 : -1;
    spos[i] = -1;
  }
  if (tid < kb) at[tid] = from[tid] = k0 + tid;
  if (tid == 0) nmove = kb;
  if (tid >= NW && tid < 16) wval[0][tid] = wval[1][tid] = -2.0, wrow[0][tid] = wrow[1][tid] = n;
  for (int c0 = 0; c0 < kb; c0 += SB) {
    const int w = min(SB, kb - c0), kc = k0 + c0;
    double a[RP][SB];
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      const int i = tid + NT * r;
#pragma unroll
      for (int q = 0; q < SB; ++q) a[r][q] = (q < w && i < n) ? A[(unsigned)(kc + q) * n + i] : 0.0;
    }
    __syncthreads();  // the previous sub-panel's lists have been read
    if (tid < w) {
      sat[tid] = sfrom[tid] = kc + tid;
      spos[kc + tid] = tid;
    }
    if (tid == 0) snmove = w;
#pragma unroll 1
    for (int q = 0; q < w; ++q) {
      const int k = kc + q;
      // pivot: max |a_ik|, i >= k (ties -> smallest i)
      double best = -1.0;
      int pr = k;
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int i = tid + NT * r;
        const double v = fabs(a[r][0]);
        if (i >= k && i < n && v > best) { best = v; pr = i; }
      }
      argmax_wave(best, pr);
      if (lane == 0) { wval[q & 1][wv] = best; wrow[q & 1][wv] = pr; }
      __syncthreads();
      best = wval[q & 1][lane & 15];
      pr = wrow[q & 1][lane & 15];
      argmax16(best, pr);
      // the owners of the pivot row and of row k publish them, and one thread notes that k and
      // pr exchange their contents
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int i = tid + NT * r;
        if (i == pr) {
#pragma unroll
          for (int j = 0; j < SB; ++j) prow[j] = a[r][j];
        }
        if (i == k && pr != k) {
#pragma unroll
          for (int j = 0; j < SB; ++j) krow[j] = a[r][j];
        }
      }
      if (tid == NT - 1 && pr != k) {
        int t = spos[pr];
        if (t < 0) {
          t = snmove++;
          sat[t] = sfrom[t] = pr;
          spos[pr] = t;
        }
        const int f = sfrom[q];
        sfrom[q] = sfrom[t];
        sfrom[t] = f;
      }
      __syncthreads();
      const double inv = 1.0 / prow[0];
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int i = tid + NT * r;
        if (i == pr && pr != k) {
#pragma unroll
          for (int j = 0; j < SB; ++j) {
            a[r][j] = krow[j];
            if (j % 8 == 7) __builtin_amdgcn_sched_barrier(0);
          }
        }
        // row k becomes the scaled pivot row, the others lose f times the pivot row
        const bool is_k = i == k;
        const double f = is_k ? -inv : a[r][0] * inv;
#pragma unroll
        for (int j = 1; j < SB; ++j) {
          a[r][j - 1] = fma(-f, prow[j], is_k ? 0.0 : a[r][j]);
          if (j % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        }
        a[r][SB - 1] = -f;
      }
    }
    // after w steps column c sits in register (c + SB - w) % SB
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      const int i = tid + NT * r;
#pragma unroll
      for (int j = 0; j < SB; ++j)
        if (j >= SB - w && i < n) A[(unsigned)(kc + j - (SB - w)) * n + i] = a[r][j];
    }
    // the sub-panel's moves, appended to the panel's: what comes to sat[e] is what the panel
    // had brought to sfrom[e]
    const int ns = snmove;
    int src = 0;
    if (tid < ns) {
      const int t = pos[sfrom[tid]];
      src = t >= 0 ? from[t] : sfrom[tid];
    }
    __syncthreads();
    if (tid < ns) {
      int t = pos[sat[tid]];
      if (t < 0) {
        t = atomicAdd(&nmove, 1);
        at[t] = sat[tid];
        pos[sat[tid]] = t;
      }
      from[t] = src;
    }
    // the panel's other columns: moves, then the rank-w update
    if (kb > w) {
      const int nc = kb - w;
      // 32-bit offsets from A: n <= 3072, n^2 < 2^24
      auto column = [&](int j) { return (unsigned)(k0 + (j < c0 ? j : j + w)) * n; };
      constexpr int UM = (2 * SB * kPanel + NT - 1) / NT;
      double v[UM];
#pragma unroll
      for (int u = 0; u < UM; ++u) {
        const int e = tid + NT * u, m = e % (2 * SB), j = e / (2 * SB);
        v[u] = m < ns && j < nc ? A[column(j) + sfrom[m]] : 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < UM; ++u) {
        const int e = tid + NT * u, m = e % (2 * SB), j = e / (2 * SB);
        if (m < ns && j < nc) A[column(j) + sat[m]] = v[u];
        // the first w moves go to the sub-panel's rows; multiplier c is in register c + SB - w
        if (j < nc) {
          if (m < w) R[j][m + SB - w] = v[u];
          else if (m < SB) R[j][m - w] = 0.0;
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int i = tid + NT * r;
        if (i >= n) continue;
        if (i >= kc && i < kc + w) {
#pragma unroll
          for (int j = 0; j < SB; ++j) a[r][j] -= i == kc + j - (SB - w) ? 1.0 : 0.0;
        }
      }
      // one column at a time, the next one's entries loaded meanwhile
      double c[RP];
#pragma unroll
      for (int r = 0; r < RP; ++r) c[r] = A[column(0) + min(tid + NT * r, n - 1)];
#pragma unroll 1
      for (int j = 0; j < nc; ++j) {
        const unsigned here = column(j), next = column(min(j + 1, nc - 1));
        double cn[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) cn[r] = A[next + min(tid + NT * r, n - 1)];
#pragma unroll
        for (int q = 0; q < SB; q += 2) {
          const double2 x = *reinterpret_cast<const double2*>(&R[j][q]);
#pragma unroll
          for (int r = 0; r < RP; ++r) c[r] = fma(a[r][q + 1], x.y, fma(a[r][q], x.x, c[r]));
          if (q % 8 == 6) __builtin_amdgcn_sched_barrier(0);  // keeps the reads of R near their use
        }
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          if (tid + NT * r < n) A[here + tid + NT * r] = c[r];
          c[r] = cn[r];
        }
      }
    }
    __syncthreads();
    if (tid < ns) spos[sat[tid]] = -1;
  }
  __syncthreads();
  const int nm = nmove;
  int old = 0;
  if (tid < nm) old = idx[from[tid]];
  __syncthreads();
  if (tid < nm) {
    idx[at[tid]] = old;
    moves[1 + tid] = at[tid];
    moves[1 + kMoves + tid] = from[tid];
  }
  if (tid == 0) moves[0] = nm;
}

typedef double d4acc __attribute__((ext_vector_type(4)));

// Columns outside the panel, JC of them per workgroup: the panel's row moves, then
// A(:, J) += (T(:, P) - I_P) A(P, J) on v_mfma_f64_16x16x4 with the columns as the product's rows, so
// that a lane's loads and stores of A run along its columns (16 lanes to 128 bytes).  The
// panel's rows of the columns sit in LDS, every wave takes 16-row tiles with the 64
// multipliers of a row in registers.
// Bound: HBM, the matrix is read and written once per 64 pivots (once per 16 before, when a
// single workgroup also made the products on the VALU).
template <int JC>
__global__ __launch_bounds__(256, 4) void k_gj_update(int n, int k0, double* __restrict__ A_all,
                                                   const int* __restrict__ ints) {
  constexpr int LS = JC + 16;  // row stride: four rows of 16 values fall in distinct bank halves
  __shared__ double R[kPanel][LS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // matrices along x: the strips of one share its multipliers in one XCD's L2
  const int s = blockIdx.x, kb = min(kPanel, n - k0), no = n - kb, j0 = blockIdx.y * JC;
  double* A = A_all + (size_t)s * n * n;
  const int* moves = ints + (size_t)s * (n + kInverseInts) + n;
  const int nm = moves[0];
  auto column = [&](int j) { return (unsigned)(j < k0 ? j : j + kb) * n; };
  // row moves, 16 columns at a time
  constexpr int UM = kMoves * 16 / 256;
#pragma unroll 1
  for (int c0 = 0; c0 < JC; c0 += 16) {
    double v[UM];
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int e = tid + 256 * u, m = e % kMoves, j = j0 + c0 + e / kMoves;
      v[u] = m < nm && j < no ? A[column(j) + moves[1 + kMoves + m]] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int e = tid + 256 * u, m = e % kMoves, j = j0 + c0 + e / kMoves;
      if (m < kPanel) R[m][c0 + e / kMoves] = m < kb ? v[u] : 0.0;  // the first kb moves go to the panel's rows
      if (m < nm && j < no) A[column(j) + moves[1 + m]] = v[u];
    }
  }
  __syncthreads();
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll 1
  for (int r0 = wv * 16; r0 < n; r0 += 64) {
    const int i = r0 + lr;
    double w[kPanel / 4];
#pragma unroll
    for (int ks = 0; ks < kPanel / 4; ++ks) {
      const int q = 4 * ks + lk;
      double t = 0.0;
      if (i < n && q < kb) t = A[(unsigned)(k0 + q) * n + i] - (i == k0 + q ? 1.0 : 0.0);
      w[ks] = t;
    }
    d4acc acc[JC / 16];
#pragma unroll
    for (int ct = 0; ct < JC / 16; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + ct * 16 + lk + 4 * e;
        acc[ct][e] = i < n && j < no ? A[column(j) + i] : 0.0;
      }
#pragma unroll
    for (int ks = 0; ks < kPanel / 4; ++ks) {
      if (ks % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // four steps of LDS reads in flight
#pragma unroll
      for (int ct = 0; ct < JC / 16; ++ct)
        acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(R[4 * ks + lk][ct * 16 + lr], w[ks], acc[ct], 0, 0, 0);
    }
#pragma unroll
    for (int ct = 0; ct < JC / 16; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + ct * 16 + lk + 4 * e;
        if (i < n && j < no) A[column(j) + i] = acc[ct][e];
      }
  }
}

// Column k goes to column idx[k]; `rows` rows of the matrix per workgroup, through LDS.
__global__ __launch_bounds__(256) void k_gj_columns(int n, int rows, double* __restrict__ A_all,
                                                    const int* __restrict__ ints) {
  extern __shared__ double strip[];  // [n][rows]
  const int s = blockIdx.y, i0 = blockIdx.x * rows, h = min(rows, n - i0);
  double* A = A_all + (size_t)s * n * n + i0;
  const int* idx = ints + (size_t)s * (n + kInverseInts);
  for (int e = threadIdx.x; e < n * rows; e += 256) {
    const int j = e / rows, i = e % rows;
    if (i < h) strip[e] = A[(size_t)j * n + i];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n * rows; e += 256) {
    const int j = e / rows, i = e % rows;
    if (i < h) A[(size_t)idx[j] * n + i] = strip[e];
  }
}

hipError_t launch_invert(int ns, int n, double* A, int* ints, hipStream_t st) {
  if (ns < 1 || n < 1 || n > 3072) return hipErrorInvalidValue;
  for (int k0 = 0; k0 < n; k0 += kPanel) {
    // sub-panels as wide as the registers hold (RP x SB doubles of the 256 VGPRs a thread of
    // 512 may use)
    if (n <= kGjThreads) k_gj_panel<1, 32><<<ns, kGjThreads, 0, st>>>(n, k0, A, ints);
    else if (n <= 2 * kGjThreads) k_gj_panel<2, 32><<<ns, kGjThreads, 0, st>>>(n, k0, A, ints);
    else if (n <= 4 * kGjThreads) k_gj_panel<4, 16><<<ns, kGjThreads, 0, st>>>(n, k0, A, ints);
    else k_gj_panel<6, 8><<<ns, kGjThreads, 0, st>>>(n, k0, A, ints);
    const int no = n - std::min(kPanel, n - k0);
    if (no == 0) continue;
    // narrow strips where the wide ones would leave CUs without a workgroup
    if ((long)ns * ((no + 31) / 32) >= 512) k_gj_update<32><<<dim3(ns, (no + 31) / 32), 256, 0, st>>>(n, k0, A, ints);
    else k_gj_update<16><<<dim3(ns, (no + 15) / 16), 256, 0, st>>>(n, k0, A, ints);
  }
  int rows = 16;
  while ((size_t)rows * n * sizeof(double) > 128 * 1024) rows /= 2;
  const size_t lds = (size_t)rows * n * sizeof(double);
  const hipError_t e =
      hipFuncSetAttribute((const void*)k_gj_columns, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  k_gj_columns<<<dim3((n + rows - 1) / rows, ns), 256, lds, st>>>(n, rows, A, ints);
  return hipGetLastError();
}

}  // namespace rbm
