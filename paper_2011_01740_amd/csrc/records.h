// The recorded maxima of a surrogate's training points (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/sur.h"

namespace ens {

constexpr int kOut = SUR_OUT;

// Records of point i, sorted (lanes past the last point repeat it).
__device__ __forceinline__ void sorted_records(const double *__restrict__ rec, int64_t n,
                                               int64_t i, double (&v)[kOut]) {
  const double *p = rec + (i < n ? i : n - 1);
#pragma unroll
  for (int j = 0; j < kOut; ++j) v[j] = p[j * n];
#pragma unroll
  for (int k = 2; k <= kOut; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
      for (int l = 0; l < kOut; ++l)
        if (!(l & j)) {
          const double a = v[l], b = v[l | j];
          const bool down = !(l & k);
          v[l] = down ? fmax(a, b) : fmin(a, b);
          v[l | j] = down ? fmin(a, b) : fmax(a, b);
        }
}

// Mean and standard deviation of the ranks (bits of `ranks`) whose spread is
// at the rounding of their logarithms, to fit[rank] and fit[kOut + rank].
hipError_t launch_rounding_spread(const double *rec, int64_t n, uint64_t ranks, double *fit,
                                  hipStream_t s);

}  // namespace ens
