// Waves per work item of the fast multipole leaf sums (k_fmm_leaf).
#pragma once
#include <algorithm>

namespace rbm {

constexpr int kFmmLeafWaves = 16;  // at most

// The expansions of an item cost about as much as this many sources.
#ifdef __HIPCC__
__host__ __device__
#endif
constexpr int fmm_far_cost(int P) { return 5 * P * P / 2; }

// N points in at most `boxes` leaves, ntask items of up to 64 targets of one leaf; far_on: expansions are
// evaluated.  4 waves where the items alone give every SIMD some (4096 items are 16 waves a SIMD), more
// below; down to a quarter of that where the work does not share out to more, as the first wave
// evaluates the expansions alone and the others would hold their place on the chip waiting for it.  Whole sums in
// us, without that bound and with it: float32 order 12, 100,000 points in 31,919 leaves 13,870 -> 12,935
// (2 waves 13,230), 71,465 in 512 1144 -> 934, 200,000 in a sheet 1294 -> 1164, 20,000 in a chain 839 -> 795;
// order 4, 30,000 points in 64 leaves 516 with 16 waves, 873 with two.
inline int fmm_leaf_waves(int N, int ntask, int boxes, int P, bool far_on) {
  int nw = ntask >= 4096 ? 4 : ntask >= 2048 ? 8 : kFmmLeafWaves;
  const int least = nw / 4;
  const double near = 27.0 * N / std::min(boxes, std::max(ntask, 1));  // sources of an item, about
  while (nw > least && nw > 1.0 + near / (far_on ? fmm_far_cost(P) : 1)) nw /= 2;
  return nw;
}

}  // namespace rbm
