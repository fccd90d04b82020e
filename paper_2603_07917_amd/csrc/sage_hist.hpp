// Binning of the neighbours' output lengths, shared by the histogram kernel
// and the dense search's select.
#pragma once
#include "sage_device.hpp"

namespace sage {

// Fixed-point scale for the weights: every fp32 weight >= 2^-20 is an integer
// multiple of 2^-43, so w * 2^43 is an exact integer; weights below 2^11 keep
// a sum of up to 256 of them below 2^63. Integer sums are order independent.
constexpr double kWeightScale = 8796093022208.0;  // 2^43

// Largest b in [0, B-1] with edges[b] <= L (0 when L < edges[0]); edges in LDS.
__device__ __forceinline__ int length_bin(const double* edges, int B, int L) {
  const double x = (double)L;
  int lo = 0, hi = B;   // invariant: edges[lo] <= x or lo == 0; the answer is < hi
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (edges[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// A neighbour's share of its bin in fixed point: its similarity, or 1.
__device__ __forceinline__ uint64_t weight_fixed(float sim, bool uniform) {
  return (uint64_t)((uniform ? 1.0 : (double)sim) * kWeightScale);
}

}  // namespace sage
