// Per-cell arithmetic of the quantum pressure and the block sums of its energy
// form, shared by the stencil kernels and the last pass of the Poisson solve.
#pragma once

#include "internal.h"

namespace fdm {

// Fixed-point form: the hardware square root and reciprocal (about 1 ulp
// each; arguments stay in the normal range, r >= the density floor), which
// keep s to a few ulp relative at every delta.  Q in FP32 is ~7 us faster
// at 256^3 than with correctly rounded sqrtf and division.
__device__ __forceinline__ float sqrt_hw(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float rcp_hw(float x) { return __builtin_amdgcn_rcpf(x); }

// FP64 square root and reciprocal for the near-empty path: the hardware
// single-precision estimate refined by two Newton steps in FP64 (relative
// error a few 1e-16 for the positive normal arguments used here), several
// times cheaper than the correctly rounded library forms.
__device__ __forceinline__ double sqrt_d(double r) {
  double y = (double)__builtin_amdgcn_rsqf((float)r);   // ~1/sqrt(r), single precision
  y = y * (1.5 - 0.5 * r * y * y);
  y = y * (1.5 - 0.5 * r * y * y);
  return r * y;
}
__device__ __forceinline__ double rcp_d(double x) {
  double y = (double)__builtin_amdgcn_rcpf((float)x);   // ~1/x, single precision
  y = y * (2.0 - x * y);
  y = y * (2.0 - x * y);
  return y;
}

// s = sqrt(R) - 1 of a cell (plain FP32 form: sqrt(R)).
template <bool FIXED>
__device__ __forceinline__ float s_of(float d, const QConst& qc) {
  const float r = 1.0f + d;
  if constexpr (FIXED) return (r >= qc.floor_f) ? d * rcp_hw(1.0f + sqrt_hw(r)) : qc.s_floor;
  return sqrtf(r >= qc.floor_f ? r : qc.floor_f);
}

// sqrt(R) of a cell in FP64 from its exact integer mass.
__device__ __forceinline__ double sqrt_r_of(long long m, const QConst& qc) {
  double r = (double)m * qc.inv_mbar;
  r = r > qc.floor_d ? r : qc.floor_d;
  return sqrt_d(r);
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  // wave64 shuffle reduction, then across the block's waves through LDS
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  __syncthreads();
  return t;
}

}  // namespace fdm
