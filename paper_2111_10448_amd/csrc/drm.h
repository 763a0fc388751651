// Entries of the Khatri-Rao DRMs of the pass's unfolding, formed on the device
// from the per-mode Gaussian factors (equation "sketch_orig").  Shared by the
// streaming sketch kernels and the partial-column kernel.
#pragma once

#include "internal.h"

namespace pstt2 {

// Psi_m(row, a) = psi_1(i_1, a) * psi_hi(h, a) for the row i_1 + n_1 h of X_m:
// psi_hi is the product of the factor entries of modes 2..m (the mixed-radix
// digits of h), multiplied in increasing mode order.
__device__ __forceinline__ double psi_hi(const SketchArgs& A, int64_t h, int a) {
  double v = 1.0;
  if (h <= 0xffffffffLL) {
    // 32-bit index arithmetic: a few instructions per division instead of the 64-bit sequence
    uint32_t r = (uint32_t)h;
    for (int q = 2; q <= A.m; ++q) {
      const uint32_t nq = (uint32_t)A.n[q - 1];
      const uint32_t iq = r % nq;
      r /= nq;
      v *= A.fac[A.psi_off[q - 1] + (int64_t)iq * A.ell + a];
    }
    return v;
  }
  int64_t r = h;
  for (int q = 2; q <= A.m; ++q) {
    const int64_t nq = A.n[q - 1];
    const int64_t iq = r % nq;
    r /= nq;
    v *= A.fac[A.psi_off[q - 1] + iq * A.ell + a];
  }
  return v;
}

// A lane's rows of Psi_m, visited in increasing order by the workgroup
// prologues: (i_1, h) with row = i_1 + n_1 h is advanced without division, and
// the caller forms psi_hi again only when h changes (and only inside the
// matrix, where h's top digit is a valid index).
struct PsiCursor {
  int64_t row = 0, h = 0, hc = -1;
  int64_t i1 = 0;
  __device__ __forceinline__ void init(const SketchArgs& A, int64_t r) {
    row = r;
    h = r / A.n[0];
    i1 = r - h * A.n[0];
  }
  __device__ __forceinline__ void advance(const SketchArgs& A, int by) {
    row += by;
    i1 += by;
    while (i1 >= A.n[0]) {
      i1 -= A.n[0];
      ++h;
    }
  }
  // true when the caller must recompute its psi_hi values for this row
  __device__ __forceinline__ bool refresh(const SketchArgs& A) {
    if (row >= A.R || A.psi_tab || h == hc) return false;
    hc = h;
    return true;
  }
  __device__ __forceinline__ double at(const SketchArgs& A, int a, double hi) const {
    if (row >= A.R || a >= A.ell) return 0.0;
    if (A.psi_tab) return A.psi_tab[row * A.L4 + a];
    return A.fac[A.psi_off[0] + i1 * A.ell + a] * hi;
  }
};

// Omega_m(gcol, c) for a global column of X_m.
__device__ __forceinline__ double omega_col(const SketchArgs& A, int64_t gcol, int c) {
  double v = 1.0;
  int64_t r = gcol;
  for (int q = A.m + 1; q <= A.d; ++q) {
    int64_t nq = A.n[q - 1];
    int64_t iq = r % nq;
    r /= nq;
    v *= A.fac[A.omega_off[q - 1] + iq * A.ell + c];
  }
  return v;
}

}  // namespace pstt2
