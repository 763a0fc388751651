// Device helpers shared by the recovery and the adjoint.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pstt2 {

// Value of v held by lane l of the wavefront (l wave-uniform), through the
// scalar unit rather than an LDS read.
__device__ __forceinline__ double lane_f64(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// W = A^{-1} for the r x r symmetric positive definite A in LDS (r <= RP <= 32), by
// one wavefront: Gauss-Jordan elimination without pivoting, lane t < 2 r holding
// column t of [A | I] in registers, the pivot column broadcast through the
// scalar unit.  Returns false when a pivot is not above 1e-26 of the largest
// diagonal entry.  (Two barriers and an LDS pass per step in a 256-thread
// workgroup took 16 us at r = 8 with the rest of the least-squares kernel.)
template <int RP, int LD>
__device__ __forceinline__ bool spd_inverse(const double (*A)[LD], int r, double (*W)[LD]) {
  const int t = threadIdx.x & 63;
  double a[RP], dmax = 0.0;
#pragma unroll
  for (int i = 0; i < RP; ++i) {
    a[i] = 0.0;
    if (i < r) {
      a[i] = t < r ? A[i][t] : (t == r + i ? 1.0 : 0.0);
      dmax = fmax(dmax, A[i][i]);
    }
  }
  bool ok = true;
#pragma unroll
  for (int k = 0; k < RP; ++k) {
    if (k < r) {   // uniform
      const double fk = lane_f64(a[k], k);
      ok = ok && fk > 1e-26 * dmax;
      const double pk = a[k] / fk;
#pragma unroll
      for (int i = 0; i < RP; ++i)
        if (i != k && i < r) a[i] -= lane_f64(a[i], k) * pk;
      a[k] = pk;
    }
  }
#pragma unroll
  for (int i = 0; i < RP; ++i)
    if (i < r && t >= r && t < 2 * r) W[i][t - r] = a[i];
  return ok;
}

}  // namespace pstt2
