// Device functions shared by the strip and the lane kernels of Lorenz-96.
#pragma once

#include <hip/hip_runtime.h>

namespace riot {
namespace {

__device__ double block_sum(double v, double *red) {
  // wave reduction then cross-wave through LDS, fixed order
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double s = 0.0;
  const int nw = (blockDim.x + 63) >> 6;
  for (int k = 0; k < nw; ++k) s += red[k];
  __syncthreads();
  return s;
}

// Workgroup-cooperative L x for one column; ext must hold n + 2w doubles of LDS
// (or be nullptr to read x from global memory with modular indexing).
__device__ void apply_L_column(int n, int w, const double *__restrict__ taps,
                               const double *__restrict__ x, double *__restrict__ y,
                               const double *__restrict__ z, int mode, double *ext) {
  if (ext) {
    for (int k = threadIdx.x; k < n + 2 * w; k += blockDim.x) {
      int src = (k - w) % n;
      if (src < 0) src += n;
      ext[k] = x[src];
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double acc;
    if (ext) {
      acc = taps[0] * ext[i + w];
      for (int dd = 1; dd <= w; ++dd) acc += taps[dd] * (ext[i + w + dd] + ext[i + w - dd]);
    } else {
      acc = taps[0] * x[i];
      for (int dd = 1; dd <= w; ++dd) {
        int ip = (i + dd) % n;
        int im = (i - dd) % n;
        if (im < 0) im += n;
        acc += taps[dd] * (x[ip] + x[im]);
      }
    }
    if (mode == 1)
      acc += z[i];
    else if (mode == 2)
      acc = (z ? z[i] : 0.0) - acc;
    y[i] = acc;
  }
  __syncthreads();
}

}  // namespace
}  // namespace riot
