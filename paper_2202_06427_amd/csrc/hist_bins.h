// hist_bins.h -- bins of a squared value against the canonical edge table
// (shared by the sweep kernels).  Not installed.
#pragma once

#include "clmap_internal.h"

namespace clm {

// ---------------------------------------------------------------- histogram bins
// Canonical bin of v against E64[0..nb] (first k with v <= E_{k+1}; v = 0 ->
// bin 0; beyond E_nb -> nb), FP64.  The edges are (k h)^2 (the last possibly
// rc^2), so the smallest m with v <= E_m is guessed from sqrt(v) / h and
// settled against the table itself: the result depends only on the table.
__device__ __forceinline__ int bin64(const double* __restrict__ E, int nb, double inv_h, double v) {
  if (!(v <= E[nb])) return nb;
  const double g = ceil(sqrt(v) * inv_h);
  int m = g > 0.0 ? (g < (double)nb ? (int)g : nb) : 0;
  while (m > 0 && v <= E[m - 1]) --m;
  while (!(v <= E[m])) ++m;  // stops at nb at the latest: v <= E_nb
  return m == 0 ? 0 : m - 1;
}

// The same with the edges in LDS and an FP32 guess: the bin is the guess's where
// its own two edges say so (10^6 particles, cutoff 12, 128 bins, FP64 form: the
// map 920 us; with the FP64 root and the table in memory 1605).
__device__ __forceinline__ int bin64_near(const double* E, int nb, float inv_h, double inv_h64, double v) {
  int k = (int)(__builtin_amdgcn_sqrtf((float)v) * inv_h);
  k = min(max(k, 0), nb - 1);
  if (__builtin_expect((v > E[k] || k == 0) && v <= E[k + 1], 1)) return k;
  return bin64(E, nb, inv_h64, v);
}

// FP32 bin with certainty flag.  The edges are formed in FP32, E_m =
// (m h)^2 for m < nb and E_nb = elast (the canonical last edge rounded to
// FP32): each is within 5 units of 2^-24 (relative) of the canonical FP64
// edge.  The bin is certain when v is farther than band from both of its
// edges; band covers the FP32 error of v plus 8 * 2^-24 * elast.
__device__ __forceinline__ float edge32(const float* Et, int m, int nb, float h, float elast) {
  if constexpr (kHistEdgeTable) return Et[m];
  const float e = (float)m * h;
  return m >= nb ? elast : e * e;
}
__device__ __forceinline__ int bin32(const float* Et, int nb, float h, float inv_h, float elast, float v,
                                     float band, bool* certain) {
  const float sq = __builtin_sqrtf(v);
  int k = (int)ceilf(sq * inv_h) - 1;
  k = k < 0 ? 0 : (k > nb ? nb : k);
  if (k < nb && k > 0 && v <= edge32(Et, k, nb, h, elast)) --k;
  else if (k < nb && v > edge32(Et, k + 1, nb, h, elast)) ++k;
  if (k >= nb) {
    *certain = (v - elast) > band;
    return nb;
  }
  const float lo = edge32(Et, k, nb, h, elast), hi = edge32(Et, k + 1, nb, h, elast);
  *certain = (k == 0 ? true : (v - lo) > band) && (hi - v) > band && v > lo && v <= hi;
  return k;
}

}  // namespace clm
