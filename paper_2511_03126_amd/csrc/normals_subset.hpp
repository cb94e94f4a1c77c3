// Which points of a cloud give k_estimate_normals the upper bound of the k-th smallest distance, and which ones a thread of its
// sweep reads.  Host and device.
#pragma once

#include <cmath>

#ifdef __HIPCC__
#define AURA_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define AURA_HOST_DEVICE inline
#endif

namespace aura {

constexpr int kNrmSubSmall = 8192, kNrmSub = 16384;
constexpr int kNrmFewCand = 1500;
constexpr int kNrmCand = 8192;    // candidates the LDS list holds (distance and index: as many words as the subset)

// `count` runs of `run` neighbouring points, run j from point j * run * stride on.
struct NrmSubset {
  int run, stride, count;
};

// n points (more than kNrmCand), k at most 256.  The list takes the points within the k-th distance of the subset, k * stride of
// them on average; a query that finds more takes several sweeps.  Half the size where they stay few.
// Runs of four cost a quarter of the cache lines, but in a cloud stored along a curve the points of a run are hardly more
// than one sample, four times as heavy: the points within the bound are then 4 * stride * Gamma(k / 4), which exceeds
// 4 * stride * (k / 4 + sqrt(24 k / 4) + 12) once in e^12 queries (the tail bound of a Gamma variable).  Where that is more than the list
// holds, single points.  150 queries on an ellipsoid stored row by row, us per call, runs everywhere / points everywhere / as
// here: 200 000 points, k = 30 45 / 54 / 45; 1 M, k = 30 148 / 168 / 148, k = 128 1653 / 176 / 163; 3 M, k = 30 4847 / 430 / 414.
AURA_HOST_DEVICE NrmSubset nrm_subset(int n, int k) {
  const int small = (n - 1) / kNrmSubSmall + 1;
  const int stride = k <= kNrmFewCand / small ? small : (n - 1) / kNrmSub + 1;
  if ((float)stride * ((float)k + sqrtf(96.0f * (float)k) + 48.0f) <= (float)kNrmCand)
    return NrmSubset{4, stride, (n / 4 - 1) / stride + 1};   // at least 1024, at most kNrmSub / 4
  return NrmSubset{1, stride, (n - 1) / stride + 1};
}

// The sweep over n points (at least 4): nrm_quads(n) quads, of which number g (at most 4 * 1024 beyond the last, for n up to
// 2^31 - 1) is read from point `first` on and adds its points but for the first `skip`: the last one may begin before its place,
// those beyond add nothing.
struct NrmQuad {
  int first, skip;
};

AURA_HOST_DEVICE int nrm_quads(int n) { return (n - 1) / 4 + 1; }

AURA_HOST_DEVICE NrmQuad nrm_quad(int g, int n) {
  const unsigned place = 4u * (unsigned)g, last = (unsigned)n - 4u;
  const unsigned first = place < last ? place : last;
  return NrmQuad{(int)first, (int)(place - first)};
}

}  // namespace aura
