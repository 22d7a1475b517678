// rbm_far_traction_static: the off-body traction sum of rbm_far_traction for callers that
// cannot allocate device memory.  Its scratch (packed sources, the split's partial sums,
// float32 copies of the targets) lives in a file-scope device array of fixed size instead of
// a context workspace, so the call needs no context and allocates nothing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <string>

#include "../../include/rbm.h"
#include "kernels.h"
#include "far_plan.h"

namespace rbm {
rbm_status set_last_error(rbm_status s, const char* msg);
}  // namespace rbm

using namespace rbm;

namespace {

constexpr int kMaxDevices = 64;

// Every GPU the library runs on holds its own copy until the process ends.
__device__ __align__(256) unsigned char scratch[kStaticBytes];

std::mutex g_mu;
unsigned char* g_scratch[kMaxDevices] = {};  // device address of `scratch`, per device

// Device address of this device's copy of `scratch`, looked up once per device with that
// device current (the name itself is a host-side stand-in, not a device address).
rbm_status scratch_address(unsigned char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return set_last_error(RBM_E_DEVICE, "device index beyond 63");
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_last_error(RBM_E_DEVICE, (std::string("hipGetSymbolAddress: ") + hipGetErrorString(e)).c_str());
    g_scratch[dev] = static_cast<unsigned char*>(p);
  }
  *out = g_scratch[dev];
  return RBM_OK;
}

}  // namespace

extern "C" rbm_status rbm_far_traction_static(int n_points, int M, const double* X, const double* Nrm,
                                              const double* q, const double* add, double* y, int precision,
                                              void* stream) {
  if (!X || !Nrm || !q || !y) return set_last_error(RBM_E_INVAL, "null argument");
  if (n_points < 1 || M < 1) return set_last_error(RBM_E_INVAL, "sizes must be >= 1");
  if (precision != 0 && precision != 1) return set_last_error(RBM_E_INVAL, "precision must be 0 or 1");
  const size_t N = (size_t)n_points;
  if (static_bytes(N, 1, precision) > kStaticOneSlot)
    return set_last_error(RBM_E_NOMEM, "more points than the static scratch takes (about 762,000 in "
                                       "float64, 838,000 in float32)");
  unsigned char* base = nullptr;
  rbm_status s = scratch_address(&base);
  if (s != RBM_OK) return s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e;
  // every unordered pair once, as in the context path, where the plan's scratch fits
  const size_t b_src = static_align(N * (precision == 0 ? 64 : 32)), b_nor = static_align(N * (precision == 0 ? 32 : 16)),
               b_out = static_align(3 * N * sizeof(double)), front = b_src + b_nor + b_out;
  if (front < kStaticBytes) {
    const SymPlan sp = sym_plan(n_points, 0, precision, std::min(sym_cap(N), (kStaticBytes - front) / sizeof(double)));
    if (sp.rows > 0) {
      void *src = base, *nor = base + b_src;
      double* sum = reinterpret_cast<double*>(base + b_src + b_nor);
      double* part = reinterpret_cast<double*>(base + front);
      if (precision == 0) {
        e = launch_pack_sources<double>(n_points, M, X, nullptr, nullptr, q, 0, Nrm, src, nor, st);
        if (e == hipSuccess) e = launch_far_sym<double>(0, sp, n_points, M, src, nor, part, sum, nullptr, st);
      } else {
        e = launch_pack_sources<float>(n_points, M, X, nullptr, nullptr, q, 0, Nrm, src, nor, st);
        if (e == hipSuccess) e = launch_far_sym<float>(0, sp, n_points, M, src, nor, part, sum, nullptr, st);
      }
      if (e == hipSuccess)
        e = launch_combine(n_points, M, 1, sum, 1.0, add, 1.0, nullptr, nullptr, 0.0, y, st);
      return e == hipSuccess ? RBM_OK : set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
    }
  }
  int split = static_split(n_points, precision);
  void* src = base;
  double* part = reinterpret_cast<double*>(base + static_align(N * (precision == 0 ? 64 : 32)));
  if (far_packing_slots(n_points) > 0) {
    split = far_packing_slots(n_points);
    if ((e = launch_far_packing(0, precision, n_points, M, X, Nrm, nullptr, nullptr, q, 0, part, st)) != hipSuccess)
      return set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
  } else if (precision == 0) {
    if ((e = launch_pack_sources<double>(n_points, M, X, nullptr, nullptr, q, 0, nullptr, src, nullptr, st)) != hipSuccess ||
        (e = launch_far<double>(0, n_points, M, X, Nrm, src, part, split, st)) != hipSuccess)
      return set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
  } else {
    unsigned char* f = reinterpret_cast<unsigned char*>(part) + static_align((size_t)split * 3 * N * sizeof(double));
    float* Xf = reinterpret_cast<float*>(f);
    float* Nf = reinterpret_cast<float*>(f + static_align(3 * N * sizeof(float)));
    if ((e = launch_cast_f32(3 * N, X, Xf, st)) != hipSuccess || (e = launch_cast_f32(3 * N, Nrm, Nf, st)) != hipSuccess ||
        (e = launch_pack_sources<float>(n_points, M, X, nullptr, nullptr, q, 0, nullptr, src, nullptr, st)) != hipSuccess ||
        (e = launch_far<float>(0, n_points, M, Xf, Nf, src, part, split, st)) != hipSuccess)
      return set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
  }
  if ((e = launch_combine(n_points, M, split, part, 1.0, add, 1.0, nullptr, nullptr, 0.0, y, st)) != hipSuccess)
    return set_last_error(RBM_E_DEVICE, hipGetErrorString(e));
  return RBM_OK;
}
