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
    if (row >= A.R || h == hc) return false;
    hc = h;
    return true;
  }
  __device__ __forceinline__ double at(const SketchArgs& A, int a, double hi) const {
    if (row >= A.R || a >= A.ell) return 0.0;
    return A.fac[A.psi_off[0] + i1 * A.ell + a] * hi;
  }
};

// The rows a workgroup prologue visits, N sketch columns a lane: values() of the current
// row.  PsiDirect forms products of m factor entries, psi_hi again as h changes.
template <int N>
struct PsiDirect {
  PsiCursor pc;
  double hi[N];
  __device__ __forceinline__ void init(const SketchArgs& A, int64_t r) { pc.init(A, r); }
  __device__ __forceinline__ void advance(const SketchArgs& A, int by) { pc.advance(A, by); }
  __device__ __forceinline__ void values(const SketchArgs& A, const int (&a)[N], double (&v)[N]) {
    if (pc.refresh(A)) {
#pragma unroll
      for (int i = 0; i < N; ++i) hi[i] = psi_hi(A, pc.h, a[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = pc.at(A, a[i], hi[i]);
  }
};

// PsiStaged reads psi_hi from a table that the workgroup forms first (psi_stage), where
// the first mode has at least kPsiStageMode entries, and PsiTable all of Psi where the
// launch has it in memory: no branch and no address that depends on a load, so a lane's
// 16 to 32 rows are loaded together.  PsiDirect made each wait for its own: 10 us before
// the first chunk, all there is to a small launch.  Values are the same.  The fields of A
// that the unrolled calls use are members: past some 300 uses of a kernel's argument
// struct the compiler copies all of it to scratch.
constexpr int kPsiStageMode = 8;
constexpr int psi_stage_size(int rows, int ell) { return (rows / kPsiStageMode + 2) * ell; }

// hi[(h - h0) ell + a] = psi_hi(h, a) for the rows [row0, row0 + rows); false: not staged.
__device__ __forceinline__ bool psi_stage(const SketchArgs& A, int64_t row0, int rows, double* hi) {
  if (A.n[0] < kPsiStageMode || row0 >= A.R) return false;
  const int64_t last = (row0 + rows < A.R ? row0 + rows : A.R) - 1;
  const int64_t h0 = row0 / A.n[0];
  const int tot = (int)(last / A.n[0] - h0 + 1) * A.ell;
  for (int e = threadIdx.x; e < tot; e += blockDim.x) hi[e] = psi_hi(A, h0 + e / A.ell, e % A.ell);
  __syncthreads();
  return true;
}

template <int N>
struct PsiStaged {
  const double *hi, *f;
  int64_t R, row;
  int n1, ell, d0, i1 = 0, h = 0;   // d0: the first row's mode-1 index
  __device__ __forceinline__ PsiStaged(const SketchArgs& A, const double* table, int64_t first_row)
      : hi(table), f(A.fac + A.psi_off[0]), R(A.R), row(first_row), n1(A.n[0]), ell(A.ell),
        d0((int)(first_row % A.n[0])) {}
  __device__ __forceinline__ void init(const SketchArgs&, int64_t r) {
    const int o = d0 + (int)(r - row);   // from the first row with the table's first h
    row = r;
    h = o / n1;
    i1 = o - h * n1;
  }
  // by at most 2 kPsiStageMode - 3: two wraps at most
  __device__ __forceinline__ void advance(const SketchArgs&, int by) {
    row += by;
    i1 += by;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool over = i1 >= n1;
      i1 -= over ? n1 : 0;
      h += over ? 1 : 0;
    }
  }
  // every lane loads (entry 0 of its row past the sketch size, table row 0 past the matrix)
  __device__ __forceinline__ void values(const SketchArgs&, const int (&a)[N], double (&v)[N]) {
    const bool in = row < R;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = a[i] < ell ? a[i] : 0;
      const double x = f[(int64_t)i1 * ell + c] * hi[(in ? h : 0) * ell + c];
      v[i] = in && a[i] < ell ? x : 0.0;
    }
  }
};

template <int N>
struct PsiTable {
  const double* tab;
  int64_t R, row = 0;
  int L4, ell;
  __device__ __forceinline__ explicit PsiTable(const SketchArgs& A) : tab(A.psi_tab), R(A.R), L4(A.L4), ell(A.ell) {}
  __device__ __forceinline__ void init(const SketchArgs&, int64_t r) { row = r; }
  __device__ __forceinline__ void advance(const SketchArgs&, int by) { row += by; }
  __device__ __forceinline__ void values(const SketchArgs&, const int (&a)[N], double (&v)[N]) {
    const bool in = row < R;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double x = tab[(in ? row : 0) * L4 + (a[i] < ell ? a[i] : 0)];
      v[i] = in && a[i] < ell ? x : 0.0;
    }
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
