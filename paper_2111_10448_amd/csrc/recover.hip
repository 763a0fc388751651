// FP64 core recovery on the GPU (paper Section 3.2 and Section 4.2).
//
//  * derive_left / derive_right: the nested Khatri-Rao DRMs share one factor per
//    mode, so S_k = X_k Omega_k follows from S_{k+1} by contracting mode k+1
//    with omega_{k+1} (block form of equation "sketch_orig"), starting from
//    Y_R = S_m; T_k = Psi_k^T X_k follows from T_{k-1} by contracting mode k
//    with psi_k, starting from T_m.
//  * basis_factor_batch / basis_form_q_batch: orthonormal bases of the sketches' ranges
//    by a column-pivoted QR (Algorithm PSTT, CPQR step).  Tall sketches are
//    first reduced by Householder TSQR (the skinny QR of Section 4.2), one
//    workgroup per 512-row block, all splits in one launch per tree
//    level; the pivots of a matrix equal the pivots of its R factor, so the
//    pivoted QR runs on the final ell x ell R.  Signs are fixed so that
//    diag(R) >= 0.  Singular values (tolerance mode) come from one-sided
//    Jacobi sweeps on the pivoted R.
//  * core_left / core_right: equation "core" and its row-space mirror.
//  * middle_z / middle_a / middle_ls: the one-pass middle core, two products and
//    a least-squares solve (Section 4.2, "PSTT2-onepass").
//  * middle_twopass: equation "PSTT2_final_core" over a slab of X.
// All temporaries are stream-ordered (hipMallocAsync), so nothing here blocks
// the host.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "internal.h"
#include "linalg.h"

namespace pstt2 {


static unsigned grid_for(int64_t n, int bs) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + bs - 1) / bs, 8192));
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---------------------------------------------------------------------------
// derived sketches
// ---------------------------------------------------------------------------
__global__ void k_derive_left(const double* __restrict__ Sin, double* __restrict__ Sout, int64_t Rk, int nk1,
                              int ell, const double* __restrict__ om) {
  const int64_t tot = Rk * ell;
  const int64_t Rk1 = Rk * nk1;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(t / Rk);
    const int64_t row = t % Rk;
    const double* sp = Sin + (int64_t)c * Rk1 + row;
    double s = 0.0;
    int i = 0;
    for (; i + 8 <= nk1; i += 8) {   // eight loads in flight, summed in order
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = sp[Rk * (i + u)];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u] * om[(i + u) * ell + c];
    }
    for (; i < nk1; ++i) s += sp[Rk * i] * om[i * ell + c];
    Sout[(int64_t)c * Rk + row] = s;
  }
}

__global__ void k_derive_right(const double* __restrict__ Tin, double* __restrict__ Tout, int64_t Ck, int nk,
                               int ell, const double* __restrict__ ps) {
  const int64_t tot = Ck * ell;
  const int64_t Cprev = Ck * nk;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(t / Ck);
    const int64_t col = t % Ck;
    const double* tp = Tin + (int64_t)a * Cprev + (int64_t)nk * col;
    double s = 0.0;
    int i = 0;
    for (; i + 8 <= nk; i += 8) {   // eight loads in flight, summed in order
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = tp[i + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += ps[(i + u) * ell + a] * v[u];
    }
    for (; i < nk; ++i) s += ps[i * ell + a] * tp[i];
    Tout[(int64_t)a * Ck + col] = s;
  }
}

hipError_t derive_left(const double* Sin, double* Sout, int64_t Rk, int nk1, int ell, const double* omega,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_derive_left, dim3(grid_for(Rk * ell, 256)), dim3(256), 0, s, Sin, Sout, Rk, nk1, ell, omega);
  return hipGetLastError();
}

hipError_t derive_right(const double* Tin, double* Tout, int64_t Ck, int nk, int ell, const double* psi,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_derive_right, dim3(grid_for(Ck * ell, 256)), dim3(256), 0, s, Tin, Tout, Ck, nk, ell, psi);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// TSQR leaves.  One workgroup factors a block of up to 512 rows by Householder
// reflections (LAPACK dlarfg convention: H = I - tau v v^T, v(j) = 1,
// beta = -sign(alpha) ||x||, tau = 0 when the column below the diagonal is already
// zero) and, from the T of the block's Q = I - V T V^T (dlarft, forward, columnwise)
// and V's top ell rows V1, the upper triangular K = T V1^T.
//
// Step j needs sigma = sum_{i>j} a_ij^2 and p_c = sum_i v_i a_ic.  With
// v_i = a_ij / (alpha - beta) below the diagonal and v_j = 1, both come from one sum
// q_c = sum_{i>j} a_ij a_ic (sigma = q_j) and row j: p_c = q_c / (alpha - beta) + a_jc.
// For c < j, where a_ic holds an earlier reflector, the same p_c is v_c . v_j, which
// T is made of.  Reflectors stay unscaled (scale in sc) until they are stored.
//
// A lane holds column 8 s + n (n = lane % 8) of set s < NS of the rows 8 i + g
// (g = lane / 8, i < QI) of its wave: column j reaches its row's lanes within the
// vector unit, a sum over rows is in registers but for three lane exchanges shared
// between the sets, and one exchange through LDS and one barrier per step remain.
// Bound by the issue of vector instructions, about half of them the multiplications:
// a level fills few compute units, and each loads and stores at some 10 bytes a
// cycle, which is why blocks are not larger.  Sixteen lanes to a column's row and 1024
// rows, or four: 43 us at ell = 20; a lane a row, two exchanges of every sum through
// LDS a step, 1024 rows: 52 us.  Now 30 us for 512 rows and 40 to 46 for 1024 at
// ell = 20 and 24 (0.8 us a step), 73 us at ell = 32 (two waves to a SIMD), 17 at ell = 12;
// 1.86 M rows at ell = 20: 270 us.
//
// V (stride M) receives the reflectors strictly below the block's diagonal and K in
// the rest of its top ell x ell; a last block of fewer than ell rows has tau = 0
// from there on, so what does not fit is not needed.
// ---------------------------------------------------------------------------
constexpr int QI = 16, QR = 8 * QI;   // rows of a lane and of a wave
// Rows of a level's blocks: 512, unless its largest matrix is one block of 1024 (40 us
// and 8 for Q at ell = 20, two levels of 512 rows 55 and 16).
static int leaf_rows(int64_t M) { return M <= 8 * QR ? 8 * QR : 4 * QR; }

// Independent problems (one per split) share each launch: workgroup g belongs
// to problem p with blk0[p] <= g < blk0[p + 1].
constexpr int MAXB = PSTT2_MAX_D;
struct LeafBatch {
  int n;
  const double* A[MAXB];
  int64_t M[MAXB];    // rows, and the stride of A's and V's columns
  double* V[MAXB];
  double* Rst[MAXB];
  int64_t ldr[MAXB];
  int qb;             // rows of a block
  double* T;          // T of the only block (L x L, L: ell rounded up), if asked for
  int64_t blk0[MAXB + 1];
};

__device__ __forceinline__ int batch_find(const int64_t* blk0, int n, int64_t g) {
  int p = 0;
  while (p + 1 < n && blk0[p + 1] <= g) ++p;
  return p;
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lanes 0..31: u summed over the halves of the wave, lanes 32..63: v
__device__ __forceinline__ double halves_sum(double u, double v) {
  const uint64_t a = __builtin_bit_cast(uint64_t, u), b = __builtin_bit_cast(uint64_t, v);
  const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
         __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}

// rows of sixteen lanes 0 and 2: u summed over the rows of the half, rows 1 and 3: v
__device__ __forceinline__ double rows_sum(double u, double v) {
  const uint64_t a = __builtin_bit_cast(uint64_t, u), b = __builtin_bit_cast(uint64_t, v);
  const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
         __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}

// v of lane J of each eight lanes
template <int J>
__device__ __forceinline__ double bcast8(double v) {
  const long u = __builtin_bit_cast(long, v);
  const long t = __builtin_amdgcn_update_dpp(0L, u, 0x150 + J, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (long)__builtin_amdgcn_update_dpp(t, u, 0x158 + J, 0xf, 0xc, false));
}

template <int NS, int QW>   // QW: most waves of a block
struct Leaf {
  static constexpr int C = 8 * NS, RS = QW + 2;
  static constexpr int L = NS == 3 ? 32 : C;   // G and T, a power of two
  double a[NS][QI];   // set (s + rd) % NS in index s after rd rounds of eight columns;
                      // wave 0's first four elements move up by one a round
  double sc[NS];      // scale of this lane's reflector
  int ell, w, n, g;
  int64_t M, rb, ldr;
  double* V;
  double* R;          // the block's R in the stack

  __device__ __forceinline__ int col(int s, int rd) const { return 8 * (s + rd < NS ? s + rd : s + rd - NS) + n; }

  // wave 0's element i, row lr < 32 of the block, once final
  __device__ __forceinline__ void put_top(int i, int lr, int rd, double (*V1)[L + 1]) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int c = col(s, rd);
      if (c < ell) {
        if (lr < ell) R[c * ldr + lr] = lr <= c ? a[s][i] : 0.0;
        if (lr > c) {
          const double v = a[s][i] * sc[s];
          if (rb + lr < M) V[c * M + rb + lr] = v;
          if (lr < L) V1[lr][c] = v;
        }
      }
    }
  }

  // Step j = 8 rd + JJ: column j is lane JJ of set 0, row j element 0 of group JJ of
  // wave 0.  red: [C][RS], of each column the waves' sums and row j; G: [j][c] =
  // v_c . v_j for c < j, tau_j at c = j.
  template <int JJ>
  __device__ __forceinline__ void step(int rd, double* red, double* G) {
    const int j = 8 * rd + JJ;
    const bool w0 = w == 0;
    double x[QI];
#pragma unroll
    for (int i = 0; i < QI; ++i) x[i] = bcast8<JJ>(a[0][i]);
    if (w0) x[0] = g > JJ ? x[0] : 0.0;   // rows up to j
    double q[NS], rj[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      double q0 = 0.0, q1 = 0.0;
#pragma unroll
      for (int i = 0; i < QI; i += 2) {
        q0 += x[i] * a[s][i];
        q1 += x[i + 1] * a[s][i + 1];
      }
      q[s] = q0 + q1;
    }
    const int row = (threadIdx.x & 63) >> 4;   // of sixteen lanes
    {   // sets by row of sixteen lanes: 0 0 0 0, 0 0 1 1, 0 2 1 2, 0 2 1 3
      const double u = halves_sum(q[0], q[NS > 1 ? 1 : 0]);
      const double v = NS > 2 ? halves_sum(q[NS > 2 ? 2 : 0], q[NS > 3 ? 3 : (NS > 2 ? 2 : 0)]) : u;
      double t = rows_sum(u, v);
      t += dpp_f64<0x128>(t);   // the two groups of a row: rotated by eight lanes
      const int st = NS == 1 ? 0 : (NS == 2 ? row >> 1 : ((row & 1) == 0 ? row >> 1 : (NS == 3 ? 2 : 2 + (row >> 1))));
      if ((g & 1) == 0) red[(8 * st + n) * RS + w] = t;
    }
    if (w0 && g == JJ) {
#pragma unroll
      for (int s = 0; s < NS; ++s) red[(8 * s + n) * RS + QW] = a[s][0];
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double* r = red + (8 * s + n) * RS;
      q[s] = (r[0] + r[1]) + (r[2] + r[3]);
      if constexpr (QW == 8) q[s] += (r[4] + r[5]) + (r[6] + r[7]);
      rj[s] = r[QW];
    }
    const double sigma = bcast8<JJ>(q[0]), alpha = bcast8<JJ>(rj[0]);
    // beta and 1 / beta by a Goldschmidt step for the root, 1 / (alpha - beta) by two
    // Newton steps, to within 2 ulp: half the operations of the root and quotients
    // rounded exactly, which every wave repeats.  |alpha - beta| >= sqrt(sigma).
    double tj = 0.0, beta = alpha, rbeta = 0.0, scal = 0.0;
    if (sigma != 0.0) {   // uniform
      const double m = alpha * alpha + sigma;
      double z, h;   // sqrt(m), half its reciprocal
      if (m >= 0x1p-900) {
        const double r0 = __builtin_amdgcn_rsq(m);
        z = m * r0;
        h = 0.5 * r0;
        const double e = __builtin_fma(-h, z, 0.5);
        z = __builtin_fma(z, e, z);
        h = __builtin_fma(h, e, h);
        z = __builtin_fma(__builtin_fma(-z, z, m), h, z);
      } else {   // residuals of the steps would be denormal
        z = sqrt(m);
        h = 0.5 / z;
      }
      beta = -copysign(z, alpha);
      const double den = alpha - beta;
      double y = __builtin_amdgcn_rcp(den);
      y = __builtin_fma(y, __builtin_fma(-den, y, 1.0), y);
      scal = __builtin_fma(y, __builtin_fma(-den, y, 1.0), y);
      h += h;
      h = __builtin_fma(h, __builtin_fma(-z, h, 1.0), h);   // 1 / sqrt(m)
      rbeta = -copysign(h, alpha);
      tj = -den * rbeta;
    }
    double p[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      p[s] = scal * q[s] + rj[s];
      if (s + rd < NS) {   // uniform; an unfinished set: a_ic -= tau scal p_c x_i, tau scal = -1 / beta
        double us = p[s] * rbeta;
        if (s == 0) us = n > JJ ? us : 0.0;
#pragma unroll
        for (int i = 0; i < QI; ++i) a[s][i] += us * x[i];
      }
    }
    if (w0) {
      if (g == 0) {   // entries c > j are not read
#pragma unroll
        for (int s = 0; s < NS; ++s) G[j * L + col(s, rd)] = s == 0 && n == JJ ? tj : sc[s] * p[s];
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double r = s == 0 && n == JJ ? beta : rj[s] - tj * p[s];
        a[s][0] = g == JJ && (s == 0 ? n >= JJ : s + rd < NS) ? r : a[s][0];
      }
    }
    if (n == JJ) sc[0] = scal;
  }
};

// Stage H of the doubling of T: of two neighbouring runs of H reflectors,
// T12 = -T1 (V1^T V2) T2.
template <int L, int H>
__device__ __forceinline__ void leaf_t(const double* G, double (*T)[L + 1], double (*X)[L / 2 + 1]) {
  if constexpr (H < L) {
    for (int e = threadIdx.x; e < L * H / 2; e += blockDim.x) {
      const int i = e % H, j = e / H % H, b1 = e / (H * H) * 2 * H, b2 = b1 + H;
      double x = 0.0;
#pragma unroll
      for (int k = 0; k < H; ++k) x += G[(b2 + k) * L + b1 + i] * T[b2 + k][b2 + j];
      X[b1 + i][j] = x;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < L * H / 2; e += blockDim.x) {
      const int i = e % H, j = e / H % H, b1 = e / (H * H) * 2 * H, b2 = b1 + H;
      double x = 0.0;
#pragma unroll
      for (int k = 0; k < H; ++k) x += T[b1 + i][b1 + k] * X[b1 + k][j];
      T[b1 + i][b2 + j] = -x;
    }
    __syncthreads();
    leaf_t<L, 2 * H>(G, T, X);
  }
}

template <int NS, int QW>
__global__ __launch_bounds__(64 * QW) void k_qr_leaf(const LeafBatch B, int ell) {
  using S_ = Leaf<NS, QW>;
  constexpr int L = S_::L, RED = S_::C * S_::RS;
  __shared__ __attribute__((aligned(16))) double red[2][RED];   // one a step: a barrier lies between its reads and its next writes
  __shared__ double G[L * L];   // G[j][c]
  __shared__ double T[L][L + 1], X[L][L / 2 + 1], V1[L][L + 1];
  const int tid = threadIdx.x;
  const int pb = batch_find(B.blk0, B.n, blockIdx.x);
  const int64_t b = blockIdx.x - B.blk0[pb];
  S_ S;
  S.ell = ell;
  S.w = __builtin_amdgcn_readfirstlane(tid >> 6);
  S.n = tid & 7;
  S.g = (tid & 63) >> 3;
  S.M = B.M[pb];
  S.rb = b * B.qb;
  S.ldr = B.ldr[pb];
  S.V = B.V[pb];
  S.R = B.Rst[pb] + b * ell;
  const int64_t wr = S.rb + QR * S.w + S.g;   // row of element 0 at first
  const bool full = S.rb + QR * (S.w + 1) <= S.M;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int c = 8 * s + S.n;
    const double* __restrict__ ac = B.A[pb] + c * S.M + wr;
    S.sc[s] = 0.0;
#pragma unroll
    for (int i = 0; i < QI; ++i) S.a[s][i] = 0.0;   // zero columns: exact no-ops
    if (c < ell) {
      if (full) {
#pragma unroll
        for (int i = 0; i < QI; ++i) S.a[s][i] = ac[8 * i];
      } else {
#pragma unroll
        for (int i = 0; i < QI; ++i)
          if (wr + 8 * i < S.M) S.a[s][i] = ac[8 * i];
      }
    }
  }
  for (int e = tid; e < 2 * RED; e += blockDim.x) (&red[0][0])[e] = 0.0;   // waves of a small block that do not run
  for (int e = tid; e < L * L; e += blockDim.x) {
    G[e] = 0.0;
    T[e / L][e % L] = 0.0;
    V1[e / L][e % L] = e / L == e % L ? 1.0 : 0.0;
  }
  __syncthreads();
  // Eight columns a round, the sets moving down by one between rounds and wave 0's top
  // rows up by one element: lane and register numbers are constants of a loop body.
  int rd = 0;
  for (; 8 * rd < ell; ++rd) {
    const int left = ell - 8 * rd;
    S.template step<0>(rd, red[0], G);
    if (left > 1) S.template step<1>(rd, red[1], G);
    if (left > 2) S.template step<2>(rd, red[0], G);
    if (left > 3) S.template step<3>(rd, red[1], G);
    if (left > 4) S.template step<4>(rd, red[0], G);
    if (left > 5) S.template step<5>(rd, red[1], G);
    if (left > 6) S.template step<6>(rd, red[0], G);
    if (left > 7) S.template step<7>(rd, red[1], G);
    if (S.w == 0) {
      S.put_top(0, 8 * rd + S.g, rd, V1);
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) S.a[s][i] = i < 3 ? S.a[s][i + 1] : 0.0;
    }
    if constexpr (NS > 1) {
#pragma unroll
      for (int i = 0; i < QI; ++i) {
        const double t = S.a[0][i];
#pragma unroll
        for (int s = 0; s + 1 < NS; ++s) S.a[s][i] = S.a[s + 1][i];
        S.a[NS - 1][i] = t;
      }
      const double t = S.sc[0];
#pragma unroll
      for (int s = 0; s + 1 < NS; ++s) S.sc[s] = S.sc[s + 1];
      S.sc[NS - 1] = t;
    }
  }
  if (S.w == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i + rd < 4) S.put_top(i, 8 * (i + rd) + S.g, rd, V1);
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int c = S.col(s, rd);
    if (c < ell) {
      double* __restrict__ vc = S.V + c * S.M + wr;
      if (S.w != 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (full || wr + 8 * i < S.M) vc[8 * i] = S.a[s][i] * S.sc[s];
      }
      if (full) {
#pragma unroll
        for (int i = 4; i < QI; ++i) vc[8 * i] = S.a[s][i] * S.sc[s];
      } else {
#pragma unroll
        for (int i = 4; i < QI; ++i)
          if (wr + 8 * i < S.M) vc[8 * i] = S.a[s][i] * S.sc[s];
      }
    }
  }
  __syncthreads();
  if (tid < L) T[tid][tid] = G[tid * L + tid];
  __syncthreads();
  leaf_t<L, 1>(G, T, X);
  for (int e = tid; e < L * L; e += blockDim.x) {
    const int i = e % L, j = e / L;
    if (B.T) B.T[e] = T[i][j];
    if (i <= j && j < ell && S.rb + i < S.M) {
      double k = 0.0;
#pragma unroll 8
      for (int u = 0; u < L; ++u) k += T[i][u] * V1[j][u];
      S.V[j * S.M + S.rb + i] = k;
    }
  }
}

// Rows of Q Z for a block's Q = I - V T V^T and Z = [Zin(b*ell .. b*ell+ell-1, :); 0]:
// Z - V (K Zin) with K = T V1^T, so a workgroup takes QA rows of a block by itself (all
// of a block's where there are many blocks): the small product in LDS, then V's rows
// against it on FP64 matrix cores.  Bound by latency (loads, small product, loads,
// stores) or, over many blocks, by memory.  The reflectors one after another, as 2 ell
// sums over the block's rows through LDS, took 41 us at ell = 24, r = 12; now 8.3 us.
// 1.86 M rows at ell = 20, r = 8: 98 -> 100 us (4.2 TB/s).
struct ApplyBatch {
  int n;
  const double* V[MAXB];
  int64_t M[MAXB];       // rows, and the stride of V's and Zout's columns
  const double* Zin[MAXB];
  int64_t ldzi[MAXB];
  int r[MAXB];
  double* Zout[MAXB];
  int qb[MAXB], parts[MAXB];   // rows of a block, workgroups that share it
  int64_t blk0[MAXB + 1];      // in workgroups
};
constexpr int QA = 128;
typedef double qr_d4 __attribute__((ext_vector_type(4)));

// CS: 16-wide tiles of the columns of Z; LP: 16 or 32, at least ell
template <int CS, int LP>
__global__ __launch_bounds__(256) void k_qr_apply(const ApplyBatch B, int ell) {
  constexpr int LD = LP + 1;
  __shared__ double Kt[LP][LD];                       // [column][row]
  __shared__ double Z[16 * CS][LD], U[16 * CS][LD];   // [column][row]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int pb = batch_find(B.blk0, B.n, blockIdx.x);
  const double* __restrict__ V = B.V[pb];
  const double* __restrict__ Zin = B.Zin[pb];
  const int64_t M = B.M[pb], ldzi = B.ldzi[pb];
  const int r = B.r[pb];
  double* __restrict__ Zout = B.Zout[pb];
  const int64_t wg = blockIdx.x - B.blk0[pb], b = wg / B.parts[pb], rb = b * B.qb[pb];
  int64_t row0 = rb + wg % B.parts[pb] * QA;
  for (int e = tid; e < LP * LP; e += 256) {
    const int c = e / LP, i = e % LP;
    Kt[c][i] = (i <= c && c < ell && rb + i < M) ? V[c * M + rb + i] : 0.0;
  }
  for (int e = tid; e < 16 * CS * LP; e += 256) {
    const int c = e / LP, i = e % LP;
    Z[c][i] = (c < r && i < ell) ? Zin[c * ldzi + b * ell + i] : 0.0;
  }
  // This wave's reflector entries of the rows at row0, the first in flight across the
  // small product.  Past the last column and row the last is read: K's rows are zero
  // there, and nothing is stored.
  double v[LP / 4][2];
  auto load = [&](int64_t row0) {
    const int64_t ra = row0 + 32 * w + l16, rb2 = ra + 16;
    const int64_t r0 = ra < M ? ra : M - 1, r1 = rb2 < M ? rb2 : M - 1;
#pragma unroll
    for (int s = 0; s < LP / 4; ++s) {
      if (4 * s < ell) {   // uniform
        const int k = 4 * s + g4;
        const double* __restrict__ vk = V + (k < ell ? k : ell - 1) * M;
        v[s][0] = vk[r0];
        v[s][1] = vk[r1];
      }
    }
    if (row0 == rb) {   // the block's top rows: unit lower triangle
#pragma unroll
      for (int s = 0; s < LP / 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int k = 4 * s + g4, lr = 32 * w + 16 * t + l16;
          v[s][t] = lr > k ? v[s][t] : (lr == k ? 1.0 : 0.0);
        }
    }
  };
  load(row0);
  __syncthreads();
  for (int e = tid; e < 16 * CS * LP; e += 256) {   // K Z
    const int c = e / LP, j = e % LP;
    double u = 0.0;
    if (c < r) {
#pragma unroll 8
      for (int k = 0; k < LP; ++k) u += Kt[k][j] * Z[c][k];
    }
    U[c][j] = u;
  }
  __syncthreads();
  const int64_t end = B.parts[pb] == 1 ? rb + B.qb[pb] : row0 + QA;
  for (;;) {
    qr_d4 acc[CS][2];
#pragma unroll
    for (int u = 0; u < CS; ++u)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[u][t] = qr_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < LP / 4; ++s) {
      if (4 * s < ell) {
#pragma unroll
        for (int u = 0; u < CS; ++u) {
          const double wk = U[16 * u + l16][4 * s + g4];
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(wk, v[s][t], acc[u][t], 0, 0, 0);
        }
      }
    }
    if (row0 + QA < end) load(row0 + QA);
#pragma unroll
    for (int u = 0; u < CS; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 16 * u + 4 * e + g4;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int64_t row = row0 + 32 * w + 16 * t + l16;
          const int lr = (int)(row - rb);
          if (c < r && row < M) Zout[c * M + row] = (lr < ell ? Z[c][lr] : 0.0) - acc[u][t][e];
        }
      }
    row0 += QA;
    if (row0 >= end) break;
  }
}

// ---- the pivoted QR of the small R factors, one wavefront per problem ----
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kXor1 = 0xB1, kXor2 = 0x4E;               // within a quad
constexpr int kHalfMirror = 0x141, kMirror = 0x140;     // within 8 and 16 lanes

// Column-pivoted QR of the ell x ell matrix R.  Lane t holds column t in
// registers; pivoting swaps positions, not data: pos is the lane's current
// column position.  Pivot: the column of largest remaining norm, first position
// on ties (norms recomputed exactly each step).  Outputs: piv (ell;
// piv[position] = original column), Qc (ell x ell, columns sign-fixed so that
// diag(R) >= 0) and, with SV, the singular values in decreasing order.
//
// A step is a chain of dependent operations of one wavefront, so the code
// shortens that chain: the column array moves up by one row per step (register
// indices stay constants without unrolling the steps), the pivot column is
// broadcast through the scalar unit, the maximum found with lane permutations
// inside the vector unit, the reflector applied unscaled while its scale (root
// and quotients) is still being formed, and the arrays shortened every eight
// steps.  ell = 24: 39 -> 22.6 us; ell = 32 with the singular values, which had a
// kernel of their own: 62 + 255 -> 156 us.
//
// Singular values by one-sided (Hestenes) Jacobi on the rows of the pivoted R
// factor, whose decreasing diagonal makes them nearly orthogonal already (about
// half the sweeps that its columns take): a round rotates E / 2 disjoint pairs
// (round-robin ordering, E = ell rounded up to even), four lanes per pair with
// eight entries each.  Sweeps end when no pair needed a rotation (at most 40).
struct CpqrBatch {
  const double* R[MAXB];
  int64_t ldr[MAXB];
  int* piv[MAXB];
  double* Qc[MAXB];
  double* sv[MAXB];
};

template <int LP, bool SV>
__global__ __launch_bounds__(64) void k_cpqr(const CpqrBatch B, int ell) {
  constexpr int VS = LP + 2;   // even row stride: 16-byte reads
  constexpr int MX = PSTT2_MAX_ELL, US = MX + 2;
  __shared__ __align__(16) double Vs[LP][VS];
  __shared__ double taus[LP], diag[LP];
  __shared__ __align__(16) double U[SV ? MX : 1][US];   // rows of the pivoted R
  const int pb = blockIdx.x;
  const double* __restrict__ R = B.R[pb];
  const int64_t ldr = B.ldr[pb];
  const int t = threadIdx.x;
  const bool act = t < ell;
  double a[LP];   // the column's rows j, j + 1, ... at step j, then zeros
#pragma unroll
  for (int i = 0; i < LP; ++i) a[i] = (act && i < ell) ? R[(int64_t)t * ldr + i] : 0.0;
  if constexpr (SV) {
    for (int i = t; i < MX * US; i += 64) (&U[0][0])[i] = 0.0;
    wave_sync();
  }
  int pos = t;
  // Steps j0 .. min(j1, ell) - 1 on arrays of N rows (the rows that can still be
  // nonzero); a finished column's array is never read again
  auto steps = [&](auto nrows, int j0, int j1) {
    constexpr int N = decltype(nrows)::value;
    for (int j = j0; j < j1 && j < ell; ++j) {
      double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 1; i < N; ++i) s4[i & 3] += a[i] * a[i];
      const double below = (s4[0] + s4[1]) + (s4[2] + s4[3]);
      const double key = (act && pos >= j) ? below + a[0] * a[0] : -1.0;
      // maximum over lanes 0..31 (the others hold -1)
      double m = key;
      m = fmax(m, dpp_f64<kXor1>(m));
      m = fmax(m, dpp_f64<kXor2>(m));
      m = fmax(m, dpp_f64<kHalfMirror>(m));
      m = fmax(m, dpp_f64<kMirror>(m));
      m = fmax(lane_f64(m, 0), lane_f64(m, 16));
      uint64_t tied = __ballot(act && pos >= j && key == m);
      if (tied == 0) tied = __ballot(act && pos == j);   // no comparable norm (NaN): no exchange
      int w = __builtin_ctzll(tied);
      while ((tied &= tied - 1) != 0) {                  // ties: the first position
        const int o = __builtin_ctzll(tied);
        if (__builtin_amdgcn_readlane(pos, o) < __builtin_amdgcn_readlane(pos, w)) w = o;
      }
      w = __builtin_amdgcn_readfirstlane(w);
      const int wpos = __builtin_amdgcn_readlane(pos, w);
      if (t == w) pos = j;
      else if (pos == j) pos = wpos;
      // pivot column (uniform) and the unscaled products with it
      double u[N], d4v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < N; ++i) u[i] = lane_f64(a[i], w);
#pragma unroll
      for (int i = 1; i < N; ++i) d4v[i & 3] += u[i] * a[i];
      const double dot = (d4v[0] + d4v[1]) + (d4v[2] + d4v[3]);
      const double sigma = lane_f64(below, w), alpha = u[0];
      double tj = 0.0, beta = alpha, scal = 0.0;
      if (sigma != 0.0) {   // uniform
        beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
        tj = (beta - alpha) / beta;
        scal = 1.0 / (alpha - beta);
      }
      // reflector j for the formation of Qc: v_0 = 1, v_i = scal u_i
      if (t == w) {
        Vs[j][0] = 1.0;
#pragma unroll
        for (int i = 1; i < N; ++i) Vs[j][i] = scal * a[i];
        taus[j] = tj;
        diag[j] = beta;
      }
      const double p = (act && pos > j) ? tj * (a[0] + scal * dot) : 0.0;
      const double top = a[0] - p;   // row j of R (the pivot's is beta)
      const double ps = p * scal;
#pragma unroll
      for (int i = 0; i + 1 < N; ++i) a[i] = a[i + 1] - ps * u[i + 1];
      a[N - 1] = 0.0;
      if constexpr (SV) {
        if (act && pos >= j) U[j][t] = t == w ? beta : top;   // by column: positions still change
      }
    }
  };
  if constexpr (LP >= 32) steps(std::integral_constant<int, 32>{}, 0, LP - 24);
  if constexpr (LP >= 24) steps(std::integral_constant<int, 24>{}, LP - 24, LP - 16);
  if constexpr (LP >= 16) steps(std::integral_constant<int, 16>{}, LP - 16, LP - 8);
  steps(std::integral_constant<int, 8>{}, LP - 8, LP);
  wave_sync();
  // Qc = H_0 ... H_{ell-1} I: lane t forms column t, sign-fixed.  At step j, q holds
  // rows j, j + 1, ... (the rows before are still the identity's)
  double q[LP];
#pragma unroll
  for (int i = 0; i < LP; ++i) q[i] = 0.0;
  auto back = [&](auto nrows, int j0, int j1) {   // steps min(j1, ell) - 1 .. j0 on N rows
    constexpr int N = decltype(nrows)::value;
    for (int j = (j1 < ell ? j1 : ell) - 1; j >= j0; --j) {
      double v[N];
#pragma unroll
      for (int i = 0; i < N; i += 2) {
        const double2 x = *(const double2*)&Vs[j][i];
        v[i] = x.x;
        v[i + 1] = x.y;
      }
      const double tj = taus[j];
#pragma unroll
      for (int i = N - 1; i > 0; --i) q[i] = q[i - 1];
      q[0] = t == j ? 1.0 : 0.0;
      double d4v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < N; ++i) d4v[i & 3] += v[i] * q[i];
      const double pd = tj * ((d4v[0] + d4v[1]) + (d4v[2] + d4v[3]));
#pragma unroll
      for (int i = 0; i < N; ++i) q[i] -= pd * v[i];
    }
  };
  back(std::integral_constant<int, 8>{}, LP - 8, LP);
  if constexpr (LP >= 16) back(std::integral_constant<int, 16>{}, LP - 16, LP - 8);
  if constexpr (LP >= 24) back(std::integral_constant<int, 24>{}, LP - 24, LP - 16);
  if constexpr (LP >= 32) back(std::integral_constant<int, 32>{}, 0, LP - 24);
  if (act) {
    const double sg = diag[t] < 0.0 ? -1.0 : 1.0;
    double* Qc = B.Qc[pb];
#pragma unroll
    for (int i = 0; i < LP; ++i)
      if (i < ell) Qc[(int64_t)t * ell + i] = sg * q[i];
    B.piv[pb][pos] = t;
  }
  if constexpr (SV) {
    const int E = (ell + 1) & ~1;
    const int pr = t >> 2, r0 = (t & 3) * 8;
    // a pair counts as orthogonal once |u_p . u_q| <= ell eps |u_p| |u_q|, the
    // rounding level of the dot product itself (a tighter test keeps rotating on
    // rounding noise and never ends before the sweep cap)
    const double tol = ell * 2.220446049250313e-16;
    wave_sync();
    for (int sweep = 0; sweep < 40; ++sweep) {
      bool any = false;
      // round rnd: pair 0 is (E - 1, rnd), pair k is (rnd + k, rnd - k) mod E - 1
      int fwd = pr, bwd = pr == 0 || pr >= E / 2 ? 0 : E - 1 - pr;
      for (int rnd = 0; rnd < E - 1; ++rnd) {
        const int x1 = pr == 0 ? E - 1 : fwd, x2 = bwd;
        fwd = fwd + 1 == E - 1 ? 0 : fwd + 1;
        bwd = bwd + 1 == E - 1 ? 0 : bwd + 1;
        const int p = x1 < x2 ? x1 : x2, q2 = x1 < x2 ? x2 : x1;
        const bool on = pr < E / 2 && q2 < ell;
        const int pp = on ? p : 0, qq = on ? q2 : 0;
        double up[8], uq[8];
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          const double2 x = *(const double2*)&U[pp][r0 + i], y = *(const double2*)&U[qq][r0 + i];
          up[i] = x.x;
          up[i + 1] = x.y;
          uq[i] = y.x;
          uq[i + 1] = y.y;
        }
        double app = 0.0, aqq = 0.0, apq = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          app += up[i] * up[i];
          aqq += uq[i] * uq[i];
          apq += up[i] * uq[i];
        }
        // the four lanes of a pair are one quad
        app += dpp_f64<kXor1>(app);
        aqq += dpp_f64<kXor1>(aqq);
        apq += dpp_f64<kXor1>(apq);
        app += dpp_f64<kXor2>(app);
        aqq += dpp_f64<kXor2>(aqq);
        apq += dpp_f64<kXor2>(apq);
        const double ab = app * aqq;
        const double lim = ab > 1e-290 ? ab * __builtin_amdgcn_rsq(ab) : sqrt(ab);
        const bool rot = on && apq != 0.0 && fabs(apq) > tol * lim;
        if (__any(rot)) {
          any = true;
          if (rot) {
            // the tangent from the approximate reciprocal and root (an inexact angle
            // leaves a residual for the next meeting), cosine and sine exact
            const double z = 0.5 * (aqq - app) * __builtin_amdgcn_rcp(apq);
            const double az = fabs(z), h = 1.0 + z * z;
            const double tg = az < 1e100 ? __builtin_amdgcn_rcp(az + h * __builtin_amdgcn_rsq(h)) : 0.0;
            const double tn = z >= 0.0 ? tg : -tg;
            const double x = 1.0 + tn * tn;
            double cs = __builtin_amdgcn_rsq(x);
            cs += 0.5 * cs * fma(-x * cs, cs, 1.0);
            cs += 0.5 * cs * fma(-x * cs, cs, 1.0);
            const double sn = cs * tn;
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
              *(double2*)&U[pp][r0 + i] = double2{cs * up[i] - sn * uq[i], cs * up[i + 1] - sn * uq[i + 1]};
              *(double2*)&U[qq][r0 + i] = double2{sn * up[i] + cs * uq[i], sn * up[i + 1] + cs * uq[i + 1]};
            }
          }
          wave_sync();
        }
      }
      if (!any) break;
    }
    wave_sync();
    // lane c < ell holds row c's norm; its place in decreasing order (ties by
    // index) is the number of rows ranked before it
    double nrm = 0.0;
    if (act)
      for (int i = 0; i < ell; ++i) nrm += U[t][i] * U[t][i];
    nrm = sqrt(nrm);
    int place = 0;
    for (int c = 0; c < ell; ++c) {
      const double o = lane_f64(nrm, c);
      place += (o > nrm || (o == nrm && c < t)) ? 1 : 0;
    }
    if (act) B.sv[pb][place] = nrm;
  }
}

struct Level {
  int64_t M;      // rows at this level
  int qb;         // rows of a block
  int64_t nb;     // blocks
  double* V;      // M x ell, reflectors and K of every block
  double* Rst;    // stacked R of this level (nb*ell x ell), input of the next level
};

struct BasisBatch {
  int n = 0, ell = 0;
  hipStream_t s = nullptr;
  std::vector<std::vector<Level>> lv;   // per problem, leaves first
  double* ws = nullptr;                 // one stream-ordered workspace for everything
  std::vector<double*> Qc, sv;
  double* tmp = nullptr;                // Q formation ping-pong buffers
};

void basis_batch_free(BasisBatch* w) {
  if (!w) return;
  if (w->ws) ws_free(w->ws, w->s);
  if (w->tmp) ws_free(w->tmp, w->s);
  delete w;
}

#define HCK(x)                         \
  do {                                 \
    hipError_t e_ = (x);               \
    if (e_ != hipSuccess) return e_;   \
  } while (0)

// As many waves as the level's largest block has rows for.
template <int QW>
static void launch_leaf(const LeafBatch& B, int64_t nblk, int64_t max_rows, int ell, hipStream_t s) {
  const dim3 g((unsigned)nblk), b(64 * (unsigned)((std::min<int64_t>(B.qb, max_rows) + QR - 1) / QR));
  if (ell <= 8) hipLaunchKernelGGL((k_qr_leaf<1, QW>), g, b, 0, s, B, ell);
  else if (ell <= 16) hipLaunchKernelGGL((k_qr_leaf<2, QW>), g, b, 0, s, B, ell);
  else if (ell <= 24) hipLaunchKernelGGL((k_qr_leaf<3, QW>), g, b, 0, s, B, ell);
  else hipLaunchKernelGGL((k_qr_leaf<4, QW>), g, b, 0, s, B, ell);
}

// Householder reflectors of the M x 16 matrix A, M <= 1024, stride M: V (strictly below
// its diagonal), T and R (16 x 16).
hipError_t qr_reflectors(const double* A, int64_t M, double* V, double* T, double* R, hipStream_t s) {
  LeafBatch B;
  std::memset(&B, 0, sizeof(B));
  B.n = 1;
  B.A[0] = A;
  B.M[0] = M;
  B.V[0] = V;
  B.Rst[0] = R;
  B.ldr[0] = 16;
  B.T = T;
  B.qb = 8 * QR;
  B.blk0[1] = 1;
  if (M <= 4 * QR) launch_leaf<4>(B, 1, M, 16, s);
  else launch_leaf<8>(B, 1, M, 16, s);
  return hipGetLastError();
}

template <bool SV>
static void launch_cpqr(const CpqrBatch& C, int n, int ell, hipStream_t s) {
  const dim3 g(n), b(64);
  if (ell <= 8) hipLaunchKernelGGL((k_cpqr<8, SV>), g, b, 0, s, C, ell);
  else if (ell <= 16) hipLaunchKernelGGL((k_cpqr<16, SV>), g, b, 0, s, C, ell);
  else if (ell <= 24) hipLaunchKernelGGL((k_cpqr<24, SV>), g, b, 0, s, C, ell);
  else hipLaunchKernelGGL((k_cpqr<32, SV>), g, b, 0, s, C, ell);
}

hipError_t basis_factor_batch(int n, const double* const* A, const int64_t* M, int ell, int* const* piv,
                              bool want_sv, BasisBatch** out, hipStream_t s) {
  BasisBatch* w = new BasisBatch();
  *out = w;
  w->n = n;
  w->ell = ell;
  w->s = s;
  w->lv.resize(n);
  // level shapes and one workspace
  int64_t tot = 0;
  int maxL = 0;
  for (std::vector<int64_t> curM(M, M + n);; ++maxL) {   // 0 rows: done
    int64_t most = 0;
    for (int p = 0; p < n; ++p) most = std::max(most, curM[p]);
    if (most == 0) break;
    for (int p = 0; p < n; ++p) {
      if (curM[p] == 0) continue;
      Level l;
      l.M = curM[p];
      l.qb = leaf_rows(most);
      l.nb = (l.M + l.qb - 1) / l.qb;
      tot += ell * l.M + l.nb * ell * ell;
      w->lv[p].push_back(l);
      curM[p] = l.nb == 1 ? 0 : l.nb * ell;
    }
  }
  tot += (int64_t)n * (ell * ell + (want_sv ? ell : 0));
  HCK(ws_alloc((void**)&w->ws, sizeof(double) * tot, s));
  double* cur = w->ws;
  w->Qc.resize(n);
  w->sv.assign(n, nullptr);
  for (int p = 0; p < n; ++p) {
    for (Level& l : w->lv[p]) {
      l.V = cur;
      cur += ell * l.M;
      l.Rst = cur;
      cur += l.nb * ell * ell;
    }
    w->Qc[p] = cur;
    cur += ell * ell;
    if (want_sv) {
      w->sv[p] = cur;
      cur += ell;
    }
  }
  // one launch per tree level over every problem that still has it
  for (int L = 0; L < maxL; ++L) {
    LeafBatch B;
    std::memset(&B, 0, sizeof(B));
    int64_t nblk = 0, max_rows = 0;
    for (int p = 0; p < n; ++p) {
      if ((int)w->lv[p].size() <= L) continue;
      const Level& l = w->lv[p][L];
      const int i = B.n++;
      B.A[i] = L == 0 ? A[p] : w->lv[p][L - 1].Rst;
      B.M[i] = l.M;
      B.V[i] = l.V;
      B.qb = l.qb;
      B.Rst[i] = l.Rst;
      B.ldr[i] = l.nb * ell;
      B.blk0[i] = nblk;
      nblk += l.nb;
      max_rows = std::max(max_rows, l.M);
    }
    B.blk0[B.n] = nblk;
    if (std::min<int64_t>(B.qb, max_rows) <= 4 * QR) launch_leaf<4>(B, nblk, max_rows, ell, s);
    else launch_leaf<8>(B, nblk, max_rows, ell, s);
    HCK(hipGetLastError());
  }
  CpqrBatch C;
  std::memset(&C, 0, sizeof(C));
  for (int p = 0; p < n; ++p) {
    C.R[p] = w->lv[p].back().Rst;
    C.ldr[p] = ell;
    C.piv[p] = piv[p];
    C.Qc[p] = w->Qc[p];
    C.sv[p] = w->sv[p];
  }
  if (want_sv) launch_cpqr<true>(C, n, ell, s);
  else launch_cpqr<false>(C, n, ell, s);
  HCK(hipGetLastError());
  return hipSuccess;
}

const double* basis_batch_sv(BasisBatch* w, int p) { return w->sv[p]; }

static void launch_apply(const ApplyBatch& B, int64_t nblk, int rmax, int ell, hipStream_t s) {
  const dim3 g((unsigned)nblk), b(256);
  if (ell <= 16) hipLaunchKernelGGL((k_qr_apply<1, 16>), g, b, 0, s, B, ell);
  else if (rmax <= 16) hipLaunchKernelGGL((k_qr_apply<1, 32>), g, b, 0, s, B, ell);
  else hipLaunchKernelGGL((k_qr_apply<2, 32>), g, b, 0, s, B, ell);
}

// Q_p (M_p x r_p) = first r_p columns of each problem's pivoted orthogonal
// factor: the reflector trees applied top-down, one launch per depth.
hipError_t basis_form_q_batch(BasisBatch* w, const int* r, double* const* Q, hipStream_t s) {
  const int n = w->n, ell = w->ell;
  int maxL = 0, rmax = 1;
  int64_t tmpsz = 0;
  std::vector<int64_t> off(n, 0);
  for (int p = 0; p < n; ++p) {
    const int L = (int)w->lv[p].size();
    maxL = std::max(maxL, L);
    rmax = std::max(rmax, r[p]);
    int64_t maxrows = 0;
    for (int i = 1; i < L; ++i) maxrows = std::max(maxrows, w->lv[p][i].M);
    off[p] = tmpsz;
    tmpsz += 2 * maxrows * r[p];
  }
  if (tmpsz > 0) HCK(ws_alloc((void**)&w->tmp, sizeof(double) * tmpsz, s));
  std::vector<const double*> zin(n);
  std::vector<int64_t> ldzi(n, ell);
  for (int p = 0; p < n; ++p) zin[p] = w->Qc[p];   // ell x r (first r columns of Qc, ld ell)
  for (int step = 0; step < maxL; ++step) {
    ApplyBatch B;
    std::memset(&B, 0, sizeof(B));
    int64_t nblk = 0, nb = 0;
    for (int p = 0; p < n; ++p) {
      const int i_l = (int)w->lv[p].size() - 1 - step;
      if (i_l >= 0) nb += w->lv[p][i_l].nb;
    }
    std::vector<std::pair<int, double*>> outs;
    for (int p = 0; p < n; ++p) {
      const int L = (int)w->lv[p].size();
      const int i_l = L - 1 - step;   // this problem's level at this depth
      if (i_l < 0) continue;
      const Level& l = w->lv[p][i_l];
      double* zout;
      if (i_l == 0) {
        zout = Q[p];
      } else {
        int64_t mr = 0;
        for (int i = 1; i < L; ++i) mr = std::max(mr, w->lv[p][i].M);
        zout = w->tmp + off[p] + (step % 2) * mr * r[p];
      }
      const int i = B.n++;
      B.V[i] = l.V;
      B.M[i] = l.M;
      B.Zin[i] = zin[p];
      B.ldzi[i] = ldzi[p];
      B.r[i] = r[p];
      B.Zout[i] = zout;
      B.qb[i] = l.qb;
      B.parts[i] = nb >= 1024 ? 1 : l.qb / QA;   // about four workgroups to a compute unit
      B.blk0[i] = nblk;
      nblk += l.nb * B.parts[i];
      outs.push_back({p, zout});
    }
    B.blk0[B.n] = nblk;
    launch_apply(B, nblk, rmax, ell, s);
    HCK(hipGetLastError());
    for (auto& o : outs) {
      const int L = (int)w->lv[o.first].size();
      zin[o.first] = o.second;
      ldzi[o.first] = w->lv[o.first][L - 1 - step].M;
    }
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// cores and the middle core's Z: batches of tall, narrow products
// ---------------------------------------------------------------------------
// G(a, i, b) = sum_{row < Rprev} Qprev(row, a) Qk(row + Rprev i, b): one product per i
hipError_t core_left(const double* Qprev, int64_t Rprev, int rprev, const double* Qk, int nk, int rk, double* G,
                     hipStream_t s) {
  return adj_gemm_tn_batch(rprev, rk, Rprev, nk, Qprev, Rprev, 1, 0, Qk, Rprev * nk, Rprev, G, (int64_t)rprev * nk,
                           rprev, s);
}

// G(a, i, b) = sum_{c < Ck} Pprev(i + nk c, a) Pk(c, b): the rows of product i are nk apart
hipError_t core_right(const double* Pprev, int64_t Cprev, int rprev, const double* Pk, int64_t Ck, int nk, int rk,
                      double* G, hipStream_t s) {
  return adj_gemm_tn_batch(rprev, rk, Ck, nk, Pprev, Cprev, nk, 1, Pk, Ck, 0, G, (int64_t)rprev * nk, rprev, s);
}

// Z(a + rp i, c) = sum_{row < Rp} Qprev(row, a) Y(row + Rp i, c);  Z is (rp nm) x ell.
hipError_t middle_z(const double* Qprev, int64_t Rprev, int rprev, const double* Y, int64_t Rm, int nm, int ell,
                    double* Z, hipStream_t s) {
  return adj_gemm_tn_batch(rprev, ell, Rprev, nm, Qprev, Rprev, 1, 0, Y, Rm, Rprev, Z, (int64_t)rprev * nm, rprev, s);
}

__global__ void k_kr_table(const double* __restrict__ fac, const KRChain ch, int64_t rows, int ell,
                           double* __restrict__ out) {
  const int64_t tot = rows * ell;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int u = (int)(t / rows);
    int64_t row = t % rows;
    double f = 1.0;
    for (int q = 0; q < ch.cnt; ++q) {
      const int64_t i = row % ch.n[q];
      row /= ch.n[q];
      f *= fac[ch.off[q] + i * ell + u];
    }
    out[t] = f;
  }
}

hipError_t kr_table(const double* fac, const KRChain& ch, int64_t rows, int ell, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_kr_table, dim3(grid_for(rows * ell, 256)), dim3(256), 0, s, fac, ch, rows, ell, out);
  return hipGetLastError();
}

__global__ void k_eye(int k, double* __restrict__ out) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < k * k; t += gridDim.x * blockDim.x)
    out[t] = (t % k == t / k) ? 1.0 : 0.0;
}

hipError_t eye(int k, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_eye, dim3(1), dim3(256), 0, s, k, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Two-sided sketches of every split in two launches.  B_k = Psi_k^T S_k
// (k < m, operand S_k = X_k Omega_k, R_k rows) or B_k = T_k Omega_k (k >= m,
// operand T_k^T, C_k rows).  A workgroup takes B.steps[p] slices of TS_ROWS
// rows of one split's operand (up to TS_STEPS, when the operand is tall
// enough to keep the CUs busy with fewer workgroups).  Per slice it stages the operand rows and the
// matching Khatri-Rao DRM rows in LDS and adds their ell x ell product into
// registers (slices in order); it writes one partial, and a wavefront per
// entry then adds a split's partials in workgroup order (deterministic).
// A DRM row is the product of the chain's factor rows; with row = i + n_0 h
// (n_0 the chain's first mode) it is psi_0(i, u) * H(h, u), where H is the
// product of the other modes' rows: a slice spans at most TS_HMAX values of
// h when n_0 >= 4, so H is formed once per h into LDS (the divisions it needs
// are per h, not per entry); smaller n_0 takes the per-entry product.
// ---------------------------------------------------------------------------
constexpr int TS_ROWS = 128;
constexpr int TS_STEPS = 8;   // slices per workgroup at most
constexpr int TS_HMAX = TS_ROWS / 4 + 2;

__device__ __forceinline__ double chain_product(const TwoSidedBatch& B, const int64_t* off, const int64_t* nmode,
                                                int q0, int j0, int cnt, int64_t rest, int u) {
  double fv = 1.0;
  if (rest <= 0xffffffffLL) {   // 32-bit index arithmetic (far fewer instructions per division)
    uint32_t r = (uint32_t)rest;
    for (int j = j0; j < cnt; ++j) {
      const uint32_t nq = (uint32_t)nmode[q0 + j];
      const uint32_t i = r % nq;
      r /= nq;
      fv *= B.fac[off[j] + (int64_t)i * B.ell + u];
    }
  } else {
    int64_t r = rest;
    for (int j = j0; j < cnt; ++j) {
      const int64_t nq = nmode[q0 + j];
      const int64_t i = r % nq;
      r /= nq;
      fv *= B.fac[off[j] + i * B.ell + u];
    }
  }
  return fv;
}

typedef double ts_d4 __attribute__((ext_vector_type(4)));

// The product on FP64 matrix cores: each wave takes 32 rows of a slice in
// 16x16x4 steps (K = 4 rows) over the output padded to 32 x 32 (four tiles).
// Lane (g, l): A operand row 4 kk + g of the first factor at column 16 a + l,
// B operand the same row of the second at column 16 b + l; tile element e
// lands at output (16 a + 4 e + g, 16 b + l).  The waves' tiles are added in
// wave order at the end.
__global__ __launch_bounds__(256) void k_two_sided_part(const TwoSidedBatch B, double* __restrict__ part) {
  __shared__ double Ss[PSTT2_MAX_ELL][TS_ROWS + 1];   // operand slice, [column][row]; reused for the wave sums
  __shared__ double Fs[PSTT2_MAX_ELL][TS_ROWS + 1];   // the slice's Khatri-Rao rows, [column][row]
  __shared__ double Hs[TS_HMAX][PSTT2_MAX_ELL + 1];
  __shared__ int32_t ri[TS_ROWS], rh[TS_ROWS];   // a slice row as i + n_0 (h0 + rh)
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6, g = lane >> 4, l = lane & 15;
  const int ell = B.ell, d = B.d;
  const int p = batch_find(B.blk0, B.n, blockIdx.x);
  const int64_t K = B.K[p];
  const int nsteps = B.steps[p];
  const int64_t r0 = (blockIdx.x - B.blk0[p]) * (int64_t)TS_ROWS * nsteps;
  const int k = B.split[p], right = B.right[p];
  const int q0 = right ? k : 0, cnt = right ? d - k : k;
  const int64_t* off = B.chain + ((int64_t)k * 2 + right) * d;
  const int64_t* nmode = B.chain + (int64_t)(d + 1) * 2 * d;
  const double* __restrict__ S = B.S[p];
  const int sc = B.scols[p] > 0 ? B.scols[p] : ell;
  const int64_t n0 = nmode[q0];
  const bool htab = n0 >= 4;
  const int nout = ell * ell;
  ts_d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[a][c] = ts_d4{0.0, 0.0, 0.0, 0.0};
  // the operand slice is loaded one slice ahead into registers: thread t
  // holds rows t % TS_ROWS of columns t / TS_ROWS + 2 j (coalesced down the rows)
  constexpr int NPRE = PSTT2_MAX_ELL * TS_ROWS / 256;
  static_assert(256 % TS_ROWS == 0 && NPRE * 256 == PSTT2_MAX_ELL * TS_ROWS, "staging layout");
  double pre[NPRE];
  auto load_slice = [&](int64_t rb) {
    const int64_t row = rb + t % TS_ROWS;
#pragma unroll
    for (int j = 0; j < NPRE; ++j) {
      const int u = t / TS_ROWS + (256 / TS_ROWS) * j;
      pre[j] = (row < K && u < sc) ? S[(int64_t)u * K + row] : 0.0;
    }
  };
  if (r0 < K) load_slice(r0);
  for (int st = 0; st < nsteps; ++st) {
    const int64_t rb = r0 + (int64_t)st * TS_ROWS;
    if (rb >= K) break;
    const int64_t h0 = rb / n0;
    __syncthreads();   // the last slice's LDS reads are done
#pragma unroll
    for (int j = 0; j < NPRE; ++j) Ss[t / TS_ROWS + (256 / TS_ROWS) * j][t % TS_ROWS] = pre[j];
    if (htab) {
      const int64_t rl = std::min<int64_t>(rb + TS_ROWS, K) - 1;
      const int nh = (int)(rl / n0 - h0 + 1);   // <= TS_ROWS / n_0 + 2 <= TS_HMAX
      for (int e = t; e < nh * ell; e += 256) {
        const int hh = e % nh, u = e / nh;
        Hs[hh][u] = chain_product(B, off, nmode, q0, 1, cnt, (h0 + hh), u);
      }
      if (t < TS_ROWS) {
        const int64_t row = rb + t, h = row / n0;
        ri[t] = (int32_t)(row - h * n0);
        rh[t] = (int32_t)(h - h0);
      }
    }
    __syncthreads();
    // the Khatri-Rao rows of the slice, all independent loads in one phase
    for (int e = t; e < PSTT2_MAX_ELL * TS_ROWS; e += 256) {
      const int r = e % TS_ROWS, u = e / TS_ROWS;
      const int64_t row = rb + r;
      double f = 0.0;
      if (row < K && u < ell)
        f = htab ? B.fac[off[0] + (int64_t)ri[r] * ell + u] * Hs[rh[r]][u]
                 : chain_product(B, off, nmode, q0, 0, cnt, row, u);
      Fs[u][r] = f;
    }
    __syncthreads();
    if (st + 1 < nsteps && rb + TS_ROWS < K) load_slice(rb + TS_ROWS);   // lands during this slice's products
#pragma unroll 2
    for (int kk = 0; kk < 8; ++kk) {
      const int r = 32 * w + 4 * kk + g;
      double f[2], sv[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        sv[a] = Ss[16 * a + l][r];
        f[a] = Fs[16 * a + l][r];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          // left: Psi_k(row, u) S_k(row, v); right: T_k(u, col) Omega_k(col, v)
          const double x = right ? sv[a] : f[a], y = right ? f[c] : sv[c];
          acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[a][c], 0, 0, 0);
        }
    }
  }
  // the four waves' tiles through LDS (Ss as scratch), added in wave order
  __syncthreads();
  double* red = &Ss[0][0];   // 4 waves x 32 x 32 doubles fit in Ss (32 x 129)
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[w * 1024 + (16 * a + 4 * e + g) * 32 + 16 * c + l] = acc[a][c][e];
  __syncthreads();
  for (int o = t; o < nout; o += 256) {
    const int u = o % ell, v = o / ell;
    double sum = red[u * 32 + v];
#pragma unroll
    for (int ww = 1; ww < 4; ++ww) sum += red[ww * 1024 + u * 32 + v];
    part[(int64_t)blockIdx.x * nout + o] = sum;
  }
}

// H(h, u) of one problem for every h, row-major (ell per row): the product of
// the factor rows of the chain's modes after the first, taken in the order
// chain_product takes them, so the values equal the per-slice table's.
// One launch for the whole batch: blockIdx.y is the problem.
__global__ void k_two_sided_htab(const TwoSidedBatch B) {
  const int p = blockIdx.y;
  const int ell = B.ell, d = B.d;
  const int k = B.split[p], right = B.right[p];
  const int q0 = right ? k : 0, cnt = right ? d - k : k;
  const int64_t* off = B.chain + ((int64_t)k * 2 + right) * d;
  const int64_t* nmode = B.chain + (int64_t)(d + 1) * 2 * d;
  const int64_t n0 = nmode[q0];
  const int64_t tot = (B.K[p] + n0 - 1) / n0 * ell;
  double* __restrict__ H = const_cast<double*>(B.H[p]);
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot; e += (int64_t)gridDim.x * blockDim.x)
    H[e] = chain_product(B, off, nmode, q0, 1, cnt, e / ell, (int)(e % ell));
}

// The same product when every problem of the batch has n_0 >= 4 and a whole H
// table (k_two_sided_htab): the next slice's operand rows, its H rows (one
// contiguous run) and each lane's first-mode factor entries are loaded into
// registers while the current slice runs on the matrix cores, and each lane
// forms its Khatri-Rao operand (first-mode factor times H) as it feeds it, so a
// slice costs two barriers and no dependent cache round trip.  Values and the
// order of every sum are those of k_two_sided_part.  FTAB: the first mode's
// factor rows (n_0 ell <= TS_FTAB entries for every problem) sit in LDS, so a
// lane keeps only their row indices, and three workgroups fit on a compute unit.
// Of the ell columns 16 NQ, and with TAIL four more, are formed: 16x16x4 tiles,
// the four on the 4x4x4 instruction, whose operands have the same lanes.  Bound by
// vector instructions around the tiles (a row's place in the first mode and H is
// carried from slice to slice, not divided out again) and the tiles' rate.
// 1.86 M rows, ell = 20: 162 -> 85 us with both; 32 columns always and a division a
// slice before.  24 and 28 columns would take two and three groups of four, 8 and 15 of
// the small instructions in place of three tiles; these were not tried.
constexpr int TS_FTAB = 1024;

template <bool FTAB, int NQ, bool TAIL>
__global__ __launch_bounds__(256, FTAB ? 3 : 2) void k_two_sided_part_h(const TwoSidedBatch B,
                                                                        double* __restrict__ part) {
  static_assert(NQ == 1 || !TAIL, "16, 20 or 32 columns");
  constexpr int W = 16 * NQ + (TAIL ? 4 : 0);   // columns formed
  constexpr int NA = NQ + (TAIL ? 1 : 0);       // operands of a lane and side
  // operand slice, [column][row]; reused for the wave sums
  __shared__ double Ss[W][TS_ROWS + 1];
  // rows of ell; columns past ell, read with the next row's, reach only outputs that are not kept
  __shared__ double Hs[(TS_HMAX + 1) * PSTT2_MAX_ELL];
  __shared__ double F1[FTAB ? TS_FTAB + PSTT2_MAX_ELL : 1];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6, g = lane >> 4, l = lane & 15;
  const int ell = B.ell, d = B.d;
  const int p = batch_find(B.blk0, B.n, blockIdx.x);
  const int64_t K = B.K[p];
  const int nsteps = B.steps[p];
  const int64_t r0 = (blockIdx.x - B.blk0[p]) * (int64_t)TS_ROWS * nsteps;
  const int k = B.split[p], right = B.right[p];
  const int q0 = right ? k : 0;
  const int64_t* off = B.chain + ((int64_t)k * 2 + right) * d;
  const int64_t* nmode = B.chain + (int64_t)(d + 1) * 2 * d;
  const double* __restrict__ S = B.S[p];
  const double* __restrict__ H = B.H[p];
  const int sc = B.scols[p] > 0 ? B.scols[p] : ell;
  const int64_t n0 = nmode[q0];
  const int64_t off0 = off[0];
  const int nout = ell * ell;
  int ucol[NA];   // this lane's columns
#pragma unroll
  for (int a = 0; a < NA; ++a) ucol[a] = a < NQ ? 16 * a + l : 16 + (lane & 3);
  if constexpr (FTAB) {
    for (int e = t; e < n0 * ell; e += 256) F1[e] = B.fac[off0 + e];   // visible after the first barrier
  }
  ts_d4 acc[NQ][NQ];
  double tx = 0.0, ty = 0.0, tt = 0.0;   // TAIL: its columns as rows, as columns, as both
#pragma unroll
  for (int a = 0; a < NQ; ++a)
#pragma unroll
    for (int c = 0; c < NQ; ++c) acc[a][c] = ts_d4{0.0, 0.0, 0.0, 0.0};
  constexpr int NPRE = W * TS_ROWS / 256;
  constexpr int NHP = (TS_HMAX * W + 255) / 256;
  double pre[NPRE], hpre[NHP];
  // lane operands: rows 32 w + 4 kk + g of the slice
  double fv[FTAB ? 1 : 2][8][NA];
  int fi[FTAB ? 2 : 1][8];   // FTAB: offset of each row's first-mode factor row in F1
  int rh[2][8];              // offset of its H row in Hs
  // first-mode index and H row of the next slice's first row, and of this lane's first
  // row in it (the H row relative to the slice's)
  const int m0 = (int)n0, dh = TS_ROWS / m0, di = TS_ROWS % m0;
  int64_t sh = r0 / m0;
  int si = (int)(r0 % m0), li = (int)((r0 + 32 * w + g) % m0), lh = (int)((r0 + 32 * w + g) / m0 - sh);
  int nhe = 0;               // entries of the loaded slice's H rows, <= TS_HMAX ell
  // the register buffer is a template argument, so every index stays static
  auto load_slice = [&](int64_t rb, auto bsel) {
    constexpr int b = decltype(bsel)::value;
    const int64_t row = rb + t % TS_ROWS;
#pragma unroll
    for (int j = 0; j < NPRE; ++j) {
      const int u = t / TS_ROWS + (256 / TS_ROWS) * j;
      pre[j] = (row < K && u < sc) ? S[(int64_t)u * K + row] : 0.0;
    }
    const int rows = (int)std::min<int64_t>(TS_ROWS, K - rb);
    nhe = (int)(((uint32_t)si + rows - 1) / (uint32_t)m0 + 1) * ell;
#pragma unroll
    for (int m = 0; m < NHP; ++m) {
      const int e = t + 256 * m;
      hpre[m] = e < nhe ? H[sh * ell + e] : 0.0;
    }
    // first-mode index and H row of each of the lane's rows (n_0 >= 4: a step
    // of four rows wraps the first mode at most once); rows past K, where S is zero,
    // take the slice's first
    int i = li, hq = lh;
    const int left = rows - 32 * w - g;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (kk > 0) {
        i += 4;
        if (i >= m0) {
          i -= m0;
          ++hq;
        }
      }
      const bool in = 4 * kk < left;
      rh[b][kk] = in ? hq * ell : 0;
      if constexpr (FTAB) {
        fi[b][kk] = in ? i * ell : 0;
      } else {
#pragma unroll
        for (int a = 0; a < NA; ++a)
          fv[b][kk][a] = (in && ucol[a] < ell) ? B.fac[off0 + (int64_t)i * ell + ucol[a]] : 0.0;
      }
    }
    sh += dh;
    if (si >= m0 - di) {   // li += di, si += di, each wrapped
      si -= m0;
      ++sh;
      --lh;
    }
    si += di;
    if (li >= m0 - di) {
      li -= m0;
      ++lh;
    }
    li += di;
  };
  auto slice = [&](int64_t rb, auto bsel) {
    constexpr int b = decltype(bsel)::value;
    __syncthreads();   // the last slice's LDS reads are done
#pragma unroll
    for (int j = 0; j < NPRE; ++j) Ss[t / TS_ROWS + (256 / TS_ROWS) * j][t % TS_ROWS] = pre[j];
#pragma unroll
    for (int m = 0; m < NHP; ++m)
      if (t + 256 * m < nhe) Hs[t + 256 * m] = hpre[m];
    __syncthreads();
    if (rb + TS_ROWS < std::min<int64_t>(K, r0 + (int64_t)TS_ROWS * nsteps)) load_slice(rb + TS_ROWS, std::integral_constant<int, b ^ 1>{});
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int r = 32 * w + 4 * kk + g;
      double x[NA], y[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const double sv = Ss[ucol[a]][r];
        const double f = (FTAB ? F1[fi[FTAB ? b : 0][kk] + ucol[a]] : fv[FTAB ? 0 : b][kk][a]) * Hs[rh[b][kk] + ucol[a]];
        // left: Psi_k(row, u) S_k(row, v); right: T_k(u, col) Omega_k(col, v)
        x[a] = right ? sv : f;
        y[a] = right ? f : sv;
      }
#pragma unroll
      for (int a = 0; a < NQ; ++a)
#pragma unroll
        for (int c = 0; c < NQ; ++c) acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], y[c], acc[a][c], 0, 0, 0);
      if constexpr (TAIL) {
        tx = __builtin_amdgcn_mfma_f64_4x4x4f64(x[NQ], y[0], tx, 0, 0, 0);
        ty = __builtin_amdgcn_mfma_f64_4x4x4f64(x[0], y[NQ], ty, 0, 0, 0);
        tt = __builtin_amdgcn_mfma_f64_4x4x4f64(x[NQ], y[NQ], tt, 0, 0, 0);
      }
    }
  };
  const std::integral_constant<int, 0> b0{};
  const std::integral_constant<int, 1> b1{};
  if (r0 < K) load_slice(r0, b0);
  int st = 0;
  for (; st + 1 < nsteps; st += 2) {
    const int64_t rb = r0 + (int64_t)st * TS_ROWS;
    if (rb >= K) break;
    slice(rb, b0);
    if (rb + TS_ROWS >= K) break;
    slice(rb + TS_ROWS, b1);
  }
  if (st + 1 == nsteps) {
    const int64_t rb = r0 + (int64_t)st * TS_ROWS;
    if (rb < K) slice(rb, b0);
  }
  __syncthreads();
  double* red = &Ss[0][0];
  static_assert(4 * W <= TS_ROWS + 1, "the four waves' W x W sums fit in Ss");
#pragma unroll
  for (int a = 0; a < NQ; ++a)
#pragma unroll
    for (int c = 0; c < NQ; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(w * W + 16 * a + 4 * e + g) * W + 16 * c + l] = acc[a][c][e];
  if constexpr (TAIL) {   // block (lane / 4) % 4 of the 4x4x4 results, element (g, lane % 4)
    const int blk = (lane >> 2) & 3, l4 = lane & 3;
    red[(w * W + 16 + g) * W + 4 * blk + l4] = tx;
    red[(w * W + 4 * blk + g) * W + 16 + l4] = ty;
    if (blk == 0) red[(w * W + 16 + g) * W + 16 + l4] = tt;
  }
  __syncthreads();
  for (int o = t; o < nout; o += 256) {
    const int u = o % ell, v = o / ell;
    double sum = red[u * W + v];
#pragma unroll
    for (int ww = 1; ww < 4; ++ww) sum += red[(ww * W + u) * W + v];
    part[(int64_t)blockIdx.x * nout + o] = sum;
  }
}

template <bool FTAB>
static void launch_part_h(const TwoSidedBatch& B, int64_t nblk, double* part, hipStream_t s) {
  const dim3 g((unsigned)nblk), b(256);
  if (B.ell <= 16) hipLaunchKernelGGL((k_two_sided_part_h<FTAB, 1, false>), g, b, 0, s, B, part);
  else if (B.ell <= 20) hipLaunchKernelGGL((k_two_sided_part_h<FTAB, 1, true>), g, b, 0, s, B, part);
  else hipLaunchKernelGGL((k_two_sided_part_h<FTAB, 2, false>), g, b, 0, s, B, part);
}

__global__ __launch_bounds__(256) void k_two_sided_sum(const TwoSidedBatch B, const double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int nout = B.ell * B.ell;
  const int64_t w = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (w >= (int64_t)B.n * nout) return;
  const int p = (int)(w / nout), o = (int)(w % nout);
  double s = 0.0;
  for (int64_t g = B.blk0[p] + lane; g < B.blk0[p + 1]; g += 64) s += part[g * nout + o];
  s = wave_sum(s);
  if (lane == 0) B.out[p][o] = s;
}

// Two-level sum for problems with many slice partials: workgroup (x, p) adds,
// for every output, the partials of its contiguous run of problem p's slices in
// slice order (threads over outputs, so the reads are coalesced), then
// k_two_sided_sum2 adds the runs in run order with the fixed butterfly.
constexpr int TS_SPLIT = 256;   // runs per problem

__global__ __launch_bounds__(256) void k_two_sided_split(const TwoSidedBatch B, const double* __restrict__ part,
                                                         double* __restrict__ runs) {
  const int p = blockIdx.y;
  const int nout = B.ell * B.ell;
  const int64_t b0 = B.blk0[p], nb = B.blk0[p + 1] - b0;
  const int64_t g0 = b0 + blockIdx.x * nb / TS_SPLIT, g1 = b0 + (blockIdx.x + 1) * nb / TS_SPLIT;
  for (int o = threadIdx.x; o < nout; o += 256) {
    double s = 0.0;
    for (int64_t g = g0; g < g1; ++g) s += part[g * nout + o];
    runs[((int64_t)p * TS_SPLIT + blockIdx.x) * nout + o] = s;
  }
}

__global__ __launch_bounds__(256) void k_two_sided_sum2(const TwoSidedBatch B, const double* __restrict__ runs) {
  const int lane = threadIdx.x & 63;
  const int nout = B.ell * B.ell;
  const int64_t w = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (w >= (int64_t)B.n * nout) return;
  const int p = (int)(w / nout), o = (int)(w % nout);
  double s = 0.0;
  for (int g = lane; g < TS_SPLIT; g += 64) s += runs[((int64_t)p * TS_SPLIT + g) * nout + o];
  s = wave_sum(s);
  if (lane == 0) B.out[p][o] = s;
}

hipError_t two_sided_batch(TwoSidedBatch& B, hipStream_t s) {
  int64_t nblk = 0;
  for (int p = 0; p < B.n; ++p) {
    B.blk0[p] = nblk;
    // several slices per workgroup only while at least 512 workgroups remain
    B.steps[p] = (int)std::max<int64_t>(1, std::min<int64_t>(TS_STEPS, B.K[p] / ((int64_t)TS_ROWS * 512)));
    const int64_t rows = (int64_t)TS_ROWS * B.steps[p];
    nblk += std::max<int64_t>(1, (B.K[p] + rows - 1) / rows);
  }
  B.blk0[B.n] = nblk;
  if (B.n == 0) return hipSuccess;
  // whole H tables when every problem's first chain mode has n_0 >= 4 (mode
  // sizes known to the caller)
  bool tab = true;
  int64_t hrows[PSTT2_MAX_D] = {};
  int64_t htot = 0;
  for (int p = 0; p < B.n && tab; ++p) {
    const int64_t n0 = B.nmode[B.right[p] ? B.split[p] : 0];
    tab = n0 >= 4;
    hrows[p] = tab ? (B.K[p] + n0 - 1) / n0 : 0;
    htot += hrows[p] * B.ell;
  }
  double* part = nullptr;
  double* htab = nullptr;
  hipError_t e = ws_alloc((void**)&part, sizeof(double) * nblk * B.ell * B.ell, s);
  if (e != hipSuccess) return e;
  if (tab) {
    e = ws_alloc((void**)&htab, sizeof(double) * std::max<int64_t>(htot, 1), s);
    if (e != hipSuccess) {
      ws_free(part, s);
      return e;
    }
    int64_t o = 0, most = 0;
    for (int p = 0; p < B.n; ++p) {
      B.H[p] = htab + o;
      o += hrows[p] * B.ell;
      most = std::max<int64_t>(most, hrows[p] * B.ell);
    }
    const unsigned gh = (unsigned)std::max<int64_t>(1, std::min<int64_t>((most + 255) / 256, 16384));
    hipLaunchKernelGGL(k_two_sided_htab, dim3(gh, (unsigned)B.n), dim3(256), 0, s, B);
    bool ftab = true;
    for (int p = 0; p < B.n; ++p) ftab = ftab && B.nmode[B.right[p] ? B.split[p] : 0] * B.ell <= TS_FTAB;
    if (ftab) launch_part_h<true>(B, nblk, part, s);
    else launch_part_h<false>(B, nblk, part, s);
  } else {
    hipLaunchKernelGGL(k_two_sided_part, dim3((unsigned)nblk), dim3(256), 0, s, B, part);
  }
  const int64_t waves = (int64_t)B.n * B.ell * B.ell;
  int64_t most = 0;
  for (int p = 0; p < B.n; ++p) most = std::max<int64_t>(most, B.blk0[p + 1] - B.blk0[p]);
  double* runs = nullptr;
  if (most >= 16 * TS_SPLIT) {
    // many slices: two levels (a wave striding over tens of thousands of
    // partials 8 ell^2 bytes apart reads one double per cache line)
    e = hipGetLastError();
    if (e == hipSuccess) e = ws_alloc((void**)&runs, sizeof(double) * B.n * TS_SPLIT * B.ell * B.ell, s);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_two_sided_split, dim3(TS_SPLIT, (unsigned)B.n), dim3(256), 0, s, B, part, runs);
      hipLaunchKernelGGL(k_two_sided_sum2, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, B, runs);
    }
  } else {
    hipLaunchKernelGGL(k_two_sided_sum, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, B, part);
  }
  if (e == hipSuccess) e = hipGetLastError();
  if (runs) ws_free(runs, s);
  if (htab) ws_free(htab, s);
  ws_free(part, s);
  return e;
}

// The value of a DRM entry as the sketch kernel used it: the FP64 product of
// factors rounded to the sketch arithmetic (FP32 for FP32 and split BF16, or
// BF16, or FP16).  The
// one-pass middle core pairs Y_R with A = P_m^T Omega_m, so both must see the
// same Omega_m.
__device__ __forceinline__ double drm_effective(double v, int prec) {
  if (prec == PSTT2_P_F64) return v;
  const float f = (float)v;
  if (prec == PSTT2_P_F16) return (double)(float)(_Float16)f;
  // split BF16 carries all 24 bits of the FP32 value in its three terms
  if (prec != PSTT2_P_BF16) return (double)f;
  uint32_t u = __float_as_uint(f);
  const uint32_t h = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return (double)__uint_as_float(h << 16);
}

// A(b, c) = sum_col Pm(col, b) Omega_m(col, c).  Every block takes a contiguous
// range of columns in 64-column tiles staged through LDS (coalesced reads of
// Pm and of the Omega_m table) and writes its r_m x ell partial; a second
// kernel adds the partials in block order (deterministic).
constexpr int MA_TILE = 64;
constexpr int MA_BLOCKS = 256;

__global__ __launch_bounds__(256) void k_middle_a_part(const double* __restrict__ Pm, int64_t Cm, int rm,
                                                       const SketchArgs G, int prec, double* __restrict__ part) {
  __shared__ double Pl[MA_TILE][PSTT2_MAX_ELL + 1];
  __shared__ double Ol[MA_TILE][PSTT2_MAX_ELL + 1];
  const int ell = G.ell;
  const int nout = rm * ell;
  const int64_t c0 = (int64_t)blockIdx.x * Cm / gridDim.x, c1 = (int64_t)(blockIdx.x + 1) * Cm / gridDim.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};   // outputs t, t + 256, t + 512, t + 768
  for (int64_t base = c0; base < c1; base += MA_TILE) {
    const int nc = (int)std::min<int64_t>(MA_TILE, c1 - base);
    __syncthreads();
    for (int i = threadIdx.x; i < MA_TILE * rm; i += blockDim.x) {
      const int j = i % MA_TILE, b = i / MA_TILE;
      Pl[j][b] = j < nc ? Pm[(int64_t)b * Cm + base + j] : 0.0;
    }
    for (int i = threadIdx.x; i < MA_TILE * G.L4; i += blockDim.x) {
      const int j = i / G.L4, c = i % G.L4;
      if (c < ell) Ol[j][c] = j < nc ? drm_effective(G.om_tab[(base + j) * G.L4 + c], prec) : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = threadIdx.x + 256 * q;
      if (t < nout) {
        const int b = t % rm, c = t / rm;
        double s = 0.0;
        for (int j = 0; j < nc; ++j) s += Pl[j][b] * Ol[j][c];
        acc[q] += s;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = threadIdx.x + 256 * q;
    if (t < nout) part[(int64_t)blockIdx.x * nout + t] = acc[q];
  }
}

// one wavefront per entry of A; lanes take partials g = lane, lane + 64, ...
// and a fixed butterfly adds them (deterministic)
__global__ __launch_bounds__(256) void k_middle_a_sum(const double* __restrict__ part, int nb, int nout,
                                                      double* __restrict__ A) {
  const int lane = threadIdx.x & 63;
  const int t = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (t >= nout) return;
  double s = 0.0;
  for (int g = lane; g < nb; g += 64) s += part[(int64_t)g * nout + t];
  s = wave_sum(s);
  if (lane == 0) A[t] = s;   // t = b + rm * c
}

hipError_t middle_a(const double* Pm, int64_t Cm, int rm, const SketchArgs& geo, int prec, double* A, hipStream_t s) {
  const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(MA_BLOCKS, (Cm + MA_TILE - 1) / MA_TILE));
  const int nout = rm * geo.ell;
  double* part = nullptr;
  hipError_t e = ws_alloc((void**)&part, sizeof(double) * nb * nout, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_middle_a_part, dim3(nb), dim3(256), 0, s, Pm, Cm, rm, geo, prec, part);
  hipLaunchKernelGGL(k_middle_a_sum, dim3((nout + 3) / 4), dim3(256), 0, s, part, nb, nout, A);
  e = hipGetLastError();
  ws_free(part, s);
  return e;
}

// Least squares min ||G A - Z||_F for G (nz x rm), A (rm x ell), Z (nz x ell),
// A of full row rank: G = Z A^+ with A^+ = A^T W, W = (A A^T)^{-1} (spd_inverse on
// the rm x rm SPD matrix A A^T); then Bm = A^T W (ell x rm) and every row of G is
// z Bm.  A is a Gaussian-like rm x ell matrix (rm < ell), so cond(A A^T) =
// cond(A)^2 stays small.  A pivot below 1e-26 of the largest diagonal (A
// numerically rank-deficient) sets flag bit 2.  Every workgroup forms the same
// small Bm (identical arithmetic) and applies it to its own rows of Z, one row
// per thread (its ell entries read once, consecutive threads on consecutive
// rows).  Latency bound: rm = 8, ell = 20: 15.5 -> 7.2 us; rm = 10, ell = 24: 22 -> 15.
template <int RP, int EP>
__global__ __launch_bounds__(256) void k_middle_ls(const double* __restrict__ Z, int64_t nz,
                                                   const double* __restrict__ A, int rm, int ell,
                                                   double* __restrict__ G, int* flag) {
  __shared__ double As[RP][EP + 1];   // A (rm x ell)
  __shared__ double Gm[RP][RP + 1];   // A A^T
  __shared__ double W[RP][RP + 1];
  __shared__ double Bm[EP][RP + 1];   // A^T W: [c][b]
  const int t = threadIdx.x;
  const int64_t rho0 = blockIdx.x * (int64_t)256 + t;
  double z[EP];   // the first row's entries, requested before the small products
#pragma unroll
  for (int c = 0; c < EP; ++c) z[c] = c < ell && rho0 < nz ? Z[(int64_t)c * nz + rho0] : 0.0;
  for (int i = t; i < rm * EP; i += 256) {
    const int a = i % rm, c = i / rm;
    As[a][c] = c < ell ? A[a + rm * c] : 0.0;
  }
  __syncthreads();
  for (int i = t; i < rm * rm; i += 256) {
    const int a = i % rm, b = i / rm;
    double sum = 0.0;
#pragma unroll
    for (int c = 0; c < EP; ++c) sum += As[a][c] * As[b][c];
    Gm[a][b] = sum;
  }
  __syncthreads();
  if (t < 64) {
    const bool ok = spd_inverse<RP>(Gm, rm, W);
    if (!ok && t == 0 && blockIdx.x == 0) atomicOr(flag, 2);
  }
  __syncthreads();
  for (int i = t; i < EP * rm; i += 256) {
    const int c = i % EP, b = i / EP;
    double sum = 0.0;
    for (int a = 0; a < rm; ++a) sum += As[a][c] * W[a][b];
    Bm[c][b] = sum;
  }
  __syncthreads();
  for (int64_t rho = rho0; rho < nz; rho += (int64_t)gridDim.x * 256) {
    if (rho != rho0) {
#pragma unroll
      for (int c = 0; c < EP; ++c) z[c] = c < ell ? Z[(int64_t)c * nz + rho] : 0.0;
    }
    for (int b = 0; b < rm; ++b) {
      double sum = 0.0;
#pragma unroll
      for (int c = 0; c < EP; ++c) sum += z[c] * Bm[c][b];
      G[rho + nz * b] = sum;
    }
  }
}

template <int RP>
static void launch_ls(const double* Z, int64_t nz, const double* A, int rm, int ell, double* G, int* flag,
                      hipStream_t s) {
  const dim3 g((unsigned)std::max<int64_t>(1, std::min<int64_t>((nz + 255) / 256, 1024))), b(256);
  if (ell <= 8) hipLaunchKernelGGL((k_middle_ls<RP, 8>), g, b, 0, s, Z, nz, A, rm, ell, G, flag);
  else if (ell <= 16) hipLaunchKernelGGL((k_middle_ls<RP, 16>), g, b, 0, s, Z, nz, A, rm, ell, G, flag);
  else if (ell <= 24) hipLaunchKernelGGL((k_middle_ls<RP, 24>), g, b, 0, s, Z, nz, A, rm, ell, G, flag);
  else hipLaunchKernelGGL((k_middle_ls<RP, 32>), g, b, 0, s, Z, nz, A, rm, ell, G, flag);
}

hipError_t middle_ls(const double* Z, int64_t nz, const double* A, int rm, int ell, double* G, int* flag,
                     hipStream_t s) {
  if (rm <= 8) launch_ls<8>(Z, nz, A, rm, ell, G, flag, s);
  else if (rm <= 16) launch_ls<16>(Z, nz, A, rm, ell, G, flag, s);
  else launch_ls<32>(Z, nz, A, rm, ell, G, flag, s);
  return hipGetLastError();
}

// Two-pass middle core over a slab of X (flat entries [first, first+count)):
// G(a, i, b) += sum Qprev(row', a) X(row' + Rp i, col') Pm(col', b).
// One block per (i, col') fibre present in the slab; FP64.  Used when X_m has a
// single column (the one-sided algorithm's last core, Pm = 1), where col' = 0
// and each block owns its own i: a block adds its fibre's share into G with a
// plain read-modify-write (slabs are applied in stream order), so the result
// is bitwise repeatable.  Otherwise the two fixed-order kernels below.
template <typename T>
__global__ __launch_bounds__(256) void k_middle_twopass(const T* __restrict__ x, int64_t first, int64_t count,
                                                        int64_t Rp, int nm, int64_t Cm, const double* __restrict__ Qp,
                                                        int rp, const double* __restrict__ Pm, int rm,
                                                        double* __restrict__ G) {
  __shared__ double red[PSTT2_MAX_ELL][4];
  __shared__ double za[PSTT2_MAX_ELL];
  const int64_t fiber0 = first / Rp;
  const int64_t f = fiber0 + blockIdx.x;              // fibre index = i + nm col'
  const int i = (int)(f % nm);
  const int64_t col = f / nm;
  const int64_t lo = std::max<int64_t>(f * Rp, first);
  const int64_t hi = std::min<int64_t>((f + 1) * Rp, first + count);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double part[PSTT2_MAX_ELL];
  for (int a = 0; a < rp; ++a) part[a] = 0.0;
  for (int64_t e = lo + threadIdx.x; e < hi; e += blockDim.x) {
    const double xv = (double)x[e - first];
    const int64_t row = e - f * Rp;
    for (int a = 0; a < rp; ++a) part[a] += Qp[(int64_t)a * Rp + row] * xv;
  }
  for (int a = 0; a < rp; ++a) {
    double v = wave_sum(part[a]);
    if (lane == 0) red[a][w] = v;
  }
  __syncthreads();
  if (threadIdx.x < rp) za[threadIdx.x] = red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3];
  __syncthreads();
  for (int t = threadIdx.x; t < rp * rm; t += blockDim.x) {
    const int a = t % rp, b = t / rp;
    G[a + (int64_t)rp * (i + (int64_t)nm * b)] += za[a] * Pm[(int64_t)b * Cm + col];
  }
}

// Two steps in a fixed order (no atomics) when X_m has more than one column:
// (1) Z = X_m(:, slab) P_m(slab, :), R_m x r_m: a thread owns one row of X_m
//     and walks its share of the slab's columns; P_m is staged row-major with
//     its rows padded to RK (Pt, zero past r_m), so a column's weights are one
//     contiguous wave-uniform read; column shares go to gj partials.
// (2) G(a, i, b) += sum_{row'} Qprev(row', a) Z(row' + R_{m-1} i, b): one block
//     per (i, b), the partials added in increasing share order.
template <typename T, int RK>
__global__ __launch_bounds__(256) void k_twopass_z(const T* __restrict__ x, int64_t first, int64_t count, int64_t R,
                                                   const double* __restrict__ Pt, int rm, int gi_count, int gj_count,
                                                   double* __restrict__ Zp) {
  const int gi = blockIdx.x % gi_count, g = blockIdx.x / gi_count;
  const int64_t row = (int64_t)gi * 256 + threadIdx.x;
  if (row >= R) return;
  const int64_t c0 = first / R, c1 = (first + count + R - 1) / R;
  const int64_t cb = c0 + g * (c1 - c0) / gj_count, ce = c0 + (g + 1) * (c1 - c0) / gj_count;
  double acc[RK];
#pragma unroll
  for (int b = 0; b < RK; ++b) acc[b] = 0.0;
  // eight columns' loads in flight; an entry outside the slab (rows of a partial
  // first or last column) reads the slab's first entry and is given weight 0
  constexpr int U = 8;
  auto load = [&](int64_t col) -> double {
    const int64_t e = col * R + row;
    const bool ok = e >= first && e < first + count;
    const double v = (double)x[ok ? e - first : 0];
    return ok ? v : 0.0;
  };
  int64_t col = cb;
  for (; col + U <= ce; col += U) {
    double xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = load(col + u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* p = Pt + (col + u) * RK;
#pragma unroll
      for (int b = 0; b < RK; ++b) acc[b] += xv[u] * p[b];
    }
  }
  for (; col < ce; ++col) {
    const double xv = load(col);
    const double* p = Pt + col * RK;
#pragma unroll
    for (int b = 0; b < RK; ++b) acc[b] += xv * p[b];
  }
#pragma unroll
  for (int b = 0; b < RK; ++b)
    if (b < rm) Zp[((int64_t)g * rm + b) * R + row] = acc[b];
}

// The same for FP64 slabs of whole columns with R even: a lane owns rows
// (2t, 2t + 1) and reads both with one 16-byte load per column.  cols are
// local to the slab (column c0 + col of X_m is x + col R).
template <int RK>
__global__ __launch_bounds__(256) void k_twopass_z2(const double* __restrict__ x, int64_t R, int64_t c0, int64_t ncol,
                                                    const double* __restrict__ Pt, int rm, int gi_count, int gj_count,
                                                    double* __restrict__ Zp) {
  const int gi = blockIdx.x % gi_count, g = blockIdx.x / gi_count;
  const int64_t row = ((int64_t)gi * 256 + threadIdx.x) * 2;
  if (row >= R) return;
  const int64_t cb = g * ncol / gj_count, ce = (g + 1) * ncol / gj_count;
  double acc0[RK], acc1[RK];
#pragma unroll
  for (int b = 0; b < RK; ++b) acc0[b] = acc1[b] = 0.0;
  constexpr int U = 8;
  int64_t col = cb;
  for (; col + U <= ce; col += U) {
    double2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *(const double2*)(x + (col + u) * R + row);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* p = Pt + (c0 + col + u) * RK;
#pragma unroll
      for (int b = 0; b < RK; ++b) {
        acc0[b] += v[u].x * p[b];
        acc1[b] += v[u].y * p[b];
      }
    }
  }
  for (; col < ce; ++col) {
    const double2 v = *(const double2*)(x + col * R + row);
    const double* p = Pt + (c0 + col) * RK;
#pragma unroll
    for (int b = 0; b < RK; ++b) {
      acc0[b] += v.x * p[b];
      acc1[b] += v.y * p[b];
    }
  }
#pragma unroll
  for (int b = 0; b < RK; ++b)
    if (b < rm) {
      Zp[((int64_t)g * rm + b) * R + row] = acc0[b];
      Zp[((int64_t)g * rm + b) * R + row + 1] = acc1[b];
    }
}

__global__ __launch_bounds__(256) void k_twopass_g(const double* __restrict__ Zp, int gj_count, int64_t Rp, int nm,
                                                   const double* __restrict__ Qp, int rp, int rm,
                                                   double* __restrict__ G) {
  constexpr int MX = PSTT2_MAX_ELL;
  __shared__ double red[MX][4];
  const int i = (int)(blockIdx.x % nm), b = (int)(blockIdx.x / nm);
  const int64_t R = Rp * nm;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double part[MX];
#pragma unroll
  for (int a = 0; a < MX; ++a) part[a] = 0.0;
  for (int64_t rr = threadIdx.x; rr < Rp; rr += blockDim.x) {
    const int64_t row = rr + Rp * i;
    double z = 0.0;
    for (int g = 0; g < gj_count; ++g) z += Zp[((int64_t)g * rm + b) * R + row];
#pragma unroll
    for (int a = 0; a < MX; ++a)
      if (a < rp) part[a] += Qp[(int64_t)a * Rp + rr] * z;
  }
#pragma unroll
  for (int a = 0; a < MX; ++a) {
    if (a < rp) {
      const double v = wave_sum(part[a]);
      if (lane == 0) red[a][w] = v;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < rp) {
    const int a = threadIdx.x;
    G[a + (int64_t)rp * (i + (int64_t)nm * b)] += red[a][0] + red[a][1] + red[a][2] + red[a][3];
  }
}

// Pt(col, b) = Pm(col, b) for b < rm, 0 for rm <= b < RK (Pt row-major, RK per row)
__global__ void k_twopass_pt(const double* __restrict__ Pm, int64_t Cm, int rm, int RK, double* __restrict__ Pt) {
  const int64_t tot = Cm * RK;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(t % RK);
    Pt[t] = b < rm ? Pm[(int64_t)b * Cm + t / RK] : 0.0;
  }
}

static int twopass_rk(int rm) { return rm <= 8 ? 8 : rm <= 16 ? 16 : rm <= 24 ? 24 : 32; }

template <typename T>
static void launch_twopass_z(const T* x, int64_t first, int64_t count, int64_t R, const double* Pt, int rm, int gi,
                             int gj, double* Zp, hipStream_t s) {
  const dim3 g((unsigned)(gi * gj)), bl(256);
  switch (twopass_rk(rm)) {
    case 8: hipLaunchKernelGGL((k_twopass_z<T, 8>), g, bl, 0, s, x, first, count, R, Pt, rm, gi, gj, Zp); break;
    case 16: hipLaunchKernelGGL((k_twopass_z<T, 16>), g, bl, 0, s, x, first, count, R, Pt, rm, gi, gj, Zp); break;
    case 24: hipLaunchKernelGGL((k_twopass_z<T, 24>), g, bl, 0, s, x, first, count, R, Pt, rm, gi, gj, Zp); break;
    default: hipLaunchKernelGGL((k_twopass_z<T, 32>), g, bl, 0, s, x, first, count, R, Pt, rm, gi, gj, Zp); break;
  }
}

hipError_t middle_twopass(int dtype, const void* x, int64_t first, int64_t count, int64_t Rprev, int nm, int64_t Cm,
                          const double* Qprev, int rprev, const double* Pm, int rm, double* G, hipStream_t s) {
  const int64_t f0 = first / Rprev;
  const int64_t f1 = (first + count + Rprev - 1) / Rprev;
  const unsigned nb = (unsigned)(f1 - f0);
  if (nb == 0) return hipSuccess;
  if (fault_take()) return hipErrorLaunchFailure;
  if (Cm > 1) {
    const int64_t R = Rprev * nm;
    const int64_t ncol = (first + count + R - 1) / R - first / R;
    // pair loads: FP64 slab of whole columns, R even, 16-byte aligned base
    const bool pair = dtype == PSTT2_F64 && R % 2 == 0 && first % R == 0 && count % R == 0 &&
                      ((uintptr_t)x % 16) == 0;
    const int gi = (int)(pair ? (R + 511) / 512 : (R + 255) / 256);
    const int gj = (int)std::max<int64_t>(1, std::min<int64_t>(ncol, 2048 / gi));
    const int RK = twopass_rk(rm);
    double *Zp = nullptr, *Pt = nullptr;
    hipError_t e = ws_alloc((void**)&Zp, sizeof(double) * gj * rm * R, s);
    if (e == hipSuccess) e = ws_alloc((void**)&Pt, sizeof(double) * Cm * RK, s);
    if (e != hipSuccess) {
      if (Zp) ws_free(Zp, s);
      return e;
    }
    hipLaunchKernelGGL(k_twopass_pt, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((Cm * RK + 255) / 256, 4096))),
                       dim3(256), 0, s, Pm, Cm, rm, RK, Pt);
    if (pair) {
      const dim3 g((unsigned)(gi * gj)), bl(256);
      const double* xd = (const double*)x;
      const int64_t c0 = first / R;
      switch (RK) {
        case 8: hipLaunchKernelGGL((k_twopass_z2<8>), g, bl, 0, s, xd, R, c0, ncol, Pt, rm, gi, gj, Zp); break;
        case 16: hipLaunchKernelGGL((k_twopass_z2<16>), g, bl, 0, s, xd, R, c0, ncol, Pt, rm, gi, gj, Zp); break;
        case 24: hipLaunchKernelGGL((k_twopass_z2<24>), g, bl, 0, s, xd, R, c0, ncol, Pt, rm, gi, gj, Zp); break;
        default: hipLaunchKernelGGL((k_twopass_z2<32>), g, bl, 0, s, xd, R, c0, ncol, Pt, rm, gi, gj, Zp); break;
      }
    } else if (dtype == PSTT2_F64) {
      launch_twopass_z((const double*)x, first, count, R, Pt, rm, gi, gj, Zp, s);
    } else {
      launch_twopass_z((const float*)x, first, count, R, Pt, rm, gi, gj, Zp, s);
    }
    hipLaunchKernelGGL(k_twopass_g, dim3((unsigned)(nm * rm)), dim3(256), 0, s, Zp, gj, Rprev, nm, Qprev, rprev, rm, G);
    e = hipGetLastError();
    ws_free(Pt, s);
    ws_free(Zp, s);
    return e;
  }
  // a single column: one fibre per i (see k_middle_twopass)
  if (nb > (unsigned)nm) return hipErrorInvalidValue;
  if (dtype == PSTT2_F64)
    hipLaunchKernelGGL(k_middle_twopass<double>, dim3(nb), dim3(256), 0, s, (const double*)x, first, count, Rprev, nm,
                       Cm, Qprev, rprev, Pm, rm, G);
  else
    hipLaunchKernelGGL(k_middle_twopass<float>, dim3(nb), dim3(256), 0, s, (const float*)x, first, count, Rprev, nm,
                       Cm, Qprev, rprev, Pm, rm, G);
  return hipGetLastError();
}

}  // namespace pstt2
