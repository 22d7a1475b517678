// Types shared by the kernels of the fast multipole far field (k_fmm.hip, k_fmm_m2l.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace rbm {

template <typename T> struct Cx { T re, im; };

// coefficient (n, m), m >= 0, of an expansion
__host__ __device__ constexpr int tri(int n, int m) { return n * (n + 1) / 2 + m; }

// Per level: points per box, first box in the expansion arrays, first workgroup of the
// level in the fused M2L launch (levels 2..L, ascending).
struct FmmLevels {
  const int* cnt[8];
  size_t off[8];
  int first[9];
};

// Float32 translations by rotation, orders 2..kFmmRotOrder (k_fmm_m2l.hip): tables of
// fmm_rotation_floats(max_level) floats for the order P and the levels 2..L, then the locals of
// those levels.
constexpr int kFmmRotOrder = 15;
size_t fmm_rotation_floats(int max_level);
hipError_t launch_fmm_rotations(int P, int L, int max_level, double D, float* tab, hipStream_t st);
hipError_t launch_fmm_m2l_rot(int P, int L, int max_level, double D, FmmLevels lv, const float* tab,
                              const Cx<float>* Mexp, Cx<float>* Lexp, hipStream_t st);

}  // namespace rbm
