// Spread of training records that are (nearly) the same at every point.  In a
// file of its own so that the dataset kernels stay where they are in theirs:
// among them, this rarely used kernel cost every fit and dataset of 262144
// points 0.7 us of 161, by the place of their code alone.
#include "records.h"

namespace {

using ens::kOut;
using ens::sorted_records;

// The ranks (bits of `ranks`) whose spread is at the rounding of their
// logarithms, as where every point has the same record: what is then taken for
// the spread, and whether there is any, is the rounding of the mean, so the order of
// the sums is part of the result.  It is 256 partial sums of the points t,
// t + 256, ..., added by a tree, of the logarithms, then of the squared
// deviations from the rounded mean.  One block per rank.  Rare: every block
// sorts every point, twice.
__global__ __launch_bounds__(256) void k_rounding_spread(const double *__restrict__ rec, int64_t n,
                                                         uint64_t ranks, double *fit) {
  __shared__ double red[256];
  const int j = blockIdx.x, t = threadIdx.x;
  if (!(ranks >> j & 1)) return;
  double mean = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    double s = 0.0;
    for (int64_t i = t; i < n; i += 256) {
      double v[kOut];
      sorted_records(rec, n, i, v);
      double x = v[0];
#pragma unroll
      for (int l = 1; l < kOut; ++l) x = l == j ? v[l] : x;
      const double d = log(x) - mean;   // pass 0: the logarithm
      s = pass == 0 ? s + d : fma(d, d, s);
    }
    red[t] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
      if (t < k) red[t] += red[t + k];
      __syncthreads();
    }
    const double total = red[0] / (double)n;
    __syncthreads();
    if (pass == 0) mean = total;
    if (t == 0) fit[pass * kOut + j] = pass == 0 ? total : sqrt(total);
  }
}

}  // namespace

namespace ens {

hipError_t launch_rounding_spread(const double *rec, int64_t n, uint64_t ranks, double *fit,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_rounding_spread, dim3(kOut), dim3(256), 0, s, rec, n, ranks, fit);
  return hipGetLastError();
}

}  // namespace ens
