// Adjoint (vector-Jacobian product) of PSTT2-onepass: X -> sketches -> cores -> X~.
//
// The one-pass approximation depends on X only through the two sketches of the
// middle unfolding, Y_R = X_m Omega_m and T_m = Psi_m^T X_m (both linear in X),
// so for a cotangent gbar of X~
//     J^T gbar = Ybar Omega_m^T + Psi_m Tbar_m        (an X_m-shaped matrix).
// The pivots and ranks of the forward pass are held fixed (they are piecewise
// constant in X).  Three phases, all on the GPU in FP64:
//   B1  one stream over gbar: core cotangents through the interface matrices
//       L_m (products G_1..G_m per row of X_m) and Rt_{m+1} (G_{m+1}..G_d per
//       column): Lbar_m = gbar_m Rt^T and Rtbar = L_m^T gbar_m come from the
//       streaming dual-contraction kernel with dense tables in place of the
//       Khatri-Rao DRMs, then a backward sweep over the interface products.
//       For the Frobenius loss, gbar = -2 (X - L_m Rt) and the stream runs over
//       X itself; the rank-r_m part enters through L_m (Rt Rt^T) and
//       Rt^T (L_m^T L_m), so the cotangent is never formed;
//   B2  back through the recovery: middle least squares, outer cores, the
//       thin QR of the pivoted sketch columns, the mode-by-mode derived sketches
//       -> (Ybar, Tbar_m);
//   B3  one stream writing J^T gbar (plus 2 (X - X~) for the fused loss).
// Derivation of the middle least-squares adjoint: with W = (A A^T)^{-1} and
// G = Z A^T W,  Zbar = Gbar W A  and
//     Abar = W Gbar^T Z - G^T Gbar W A - W Gbar^T G A.
// Thin QR B = Q R (diag R > 0) with cotangent Qbar only:
//     Bbar = (Qbar + Q copyltu(M)) R^{-T},  M = -Qbar^T Q,
// where copyltu(M) mirrors the lower triangle of M onto the upper one.
#include <algorithm>
#include <cstring>

#include "internal.h"
#include "linalg.h"

namespace pstt2 {

static unsigned grid_for(int64_t n, int bs) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + bs - 1) / bs, 8192));
}

__device__ __forceinline__ double wsum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// out[i * L4 + c] = in[i * si + c * sc] for c < cnt, 0 for cnt <= c < L4 (i < rows)
__global__ void k_table(const double* __restrict__ in, int64_t rows, int cnt, int64_t si, int64_t sc, int L4,
                        double* __restrict__ out) {
  const int64_t tot = rows * L4;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t / L4;
    const int c = (int)(t % L4);
    out[t] = c < cnt ? in[i * si + c * sc] : 0.0;
  }
}

// B (rows x cols) = A^T for A cols x rows, both column-major
__global__ void k_transpose(const double* __restrict__ A, int64_t arows, int64_t acols, double* __restrict__ B) {
  const int64_t tot = arows * acols;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = t % acols, i = t / acols;   // B(j, i) = A(i, j)
    B[j + acols * i] = A[i + arows * j];
  }
}

// Y += alpha X (n entries)
__global__ void k_axpy(int64_t n, double alpha, const double* __restrict__ X, double* __restrict__ Y) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    Y[t] += alpha * X[t];
}

// ---- middle least-squares adjoint (one workgroup; p = r_{m-1} n_m rows) ----
// G (p x r), Gbar (p x r), Z (p x ell), A (r x ell) -> Zbar (p x ell), Abar (r x ell).
// Latency bound: sixteen wavefronts (the first inverts A A^T while the others
// form the products over p, four entries each in flight).  With four wavefronts
// and one entry at a time it took 60 us at p = 192, r = 8, ell = 20; now 21.
template <int RP>
__global__ __launch_bounds__(1024) void k_ls_adjoint(const double* __restrict__ G, const double* __restrict__ Gb,
                                                     const double* __restrict__ Z, const double* __restrict__ A,
                                                     int64_t p, int r, int ell, double* __restrict__ Zb,
                                                     double* __restrict__ Ab) {
  constexpr int MX = PSTT2_MAX_ELL;
  __shared__ double AAt[RP][RP + 1];
  __shared__ double Wm[RP][RP + 1];    // (A A^T)^{-1}
  __shared__ double WE[RP][RP + 1];    // W E^T
  __shared__ double As[RP][MX + 1];    // A (r x ell)
  __shared__ double WA[RP][MX + 1];    // W A (r x ell)
  __shared__ double GbZ[RP][MX + 1];   // Gbar^T Z (r x ell)
  __shared__ double E[RP][RP + 1];     // G^T Gbar (r x r)
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  for (int i = t; i < r * ell; i += 1024) As[i % r][i / r] = A[i];
  __syncthreads();
  for (int i = t; i < r * r; i += 1024) {
    const int a = i % r, b = i / r;
    double s = 0.0;
    for (int c = 0; c < ell; ++c) s += As[a][c] * As[b][c];
    AAt[a][b] = s;
  }
  __syncthreads();
  if (wv == 0) {
    (void)spd_inverse<RP>(AAt, r, Wm);
  } else {
    // Gbar^T Z and G^T Gbar, a wavefront per entry
    const int n = r * ell + r * r;
    for (int i0 = 4 * (wv - 1); i0 < n; i0 += 60) {
      const double *x[4], *y[4];
      double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u < n ? i0 + u : n - 1;
        if (i < r * ell) {
          x[u] = Gb + (int64_t)(i % r) * p;
          y[u] = Z + (int64_t)(i / r) * p;
        } else {
          const int j = i - r * ell;
          x[u] = G + (int64_t)(j % r) * p;
          y[u] = Gb + (int64_t)(j / r) * p;
        }
      }
      for (int64_t q = lane; q < p; q += 64)
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] += x[u][q] * y[u][q];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s[u] = wsum(s[u]);
        const int i = i0 + u;
        if (lane == 0 && i < n) {
          if (i < r * ell) GbZ[i % r][i / r] = s[u];
          else E[(i - r * ell) % r][(i - r * ell) / r] = s[u];
        }
      }
    }
  }
  __syncthreads();
  for (int i = t; i < r * (ell + r); i += 1024) {
    const int a = i % r, c = i / r;
    double s = 0.0;
    if (c < ell) {
      for (int b = 0; b < r; ++b) s += Wm[a][b] * As[b][c];
      WA[a][c] = s;
    } else {
      for (int k = 0; k < r; ++k) s += Wm[a][k] * E[c - ell][k];
      WE[a][c - ell] = s;
    }
  }
  __syncthreads();
  // Zbar = Gbar (W A)
  for (int64_t i = t; i < p * ell; i += 1024) {
    const int64_t q = i % p;
    const int c = (int)(i / p);
    double s = 0.0;
    for (int b = 0; b < r; ++b) s += Gb[(int64_t)b * p + q] * WA[b][c];
    Zb[i] = s;
  }
  // Abar = W (Gbar^T Z) - E (W A) - W E^T A
  for (int i = t; i < r * ell; i += 1024) {
    const int a = i % r, c = i / r;
    double s = 0.0;
    for (int b = 0; b < r; ++b) s += Wm[a][b] * GbZ[b][c] - E[a][b] * WA[b][c] - WE[a][b] * As[b][c];
    Ab[i] = s;
  }
}

// ---- right outer cores: G_k(a, i, b) = sum_c Pp(i + nk c, a) Pk(c, b) ----
// Ppbar(i + nk c, a) += sum_b Gbar(a, i, b) Pk(c, b)
__global__ void k_core_right_adj_prev(const double* __restrict__ Gb, const double* __restrict__ Pk, int64_t Ck, int nk,
                                      int rp, int rk, double* __restrict__ Ppb) {
  const int64_t Cp = Ck * nk;
  const int64_t tot = Cp * rp;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rowp = t % Cp;
    const int a = (int)(t / Cp);
    const int i = (int)(rowp % nk);
    const int64_t c = rowp / nk;
    double s = 0.0;
    for (int b = 0; b < rk; ++b) s += Gb[a + (int64_t)rp * (i + (int64_t)nk * b)] * Pk[(int64_t)b * Ck + c];
    Ppb[t] += s;
  }
}
// Pkbar(c, b) += sum_{a, i} Gbar(a, i, b) Pp(i + nk c, a), one wavefront per entry
// (few entries: one thread each over rp nk dependent loads took 44 us at 48 x 6
// entries of 288 terms, now 5)
__global__ __launch_bounds__(256) void k_core_right_adj_next(const double* __restrict__ Gb, const double* __restrict__ Pp,
                                                             int64_t Ck, int nk, int rp, int rk,
                                                             double* __restrict__ Pkb) {
  const int lane = threadIdx.x & 63;
  const int64_t Cp = Ck * nk, tot = Ck * rk;
  for (int64_t t = (blockIdx.x * (int64_t)256 + threadIdx.x) >> 6; t < tot; t += ((int64_t)gridDim.x * 256) >> 6) {
    const int64_t c = t % Ck;
    const int b = (int)(t / Ck);
    double s = 0.0;
    for (int e = lane; e < rp * nk; e += 64) {
      const int a = e / nk, i = e - a * nk;
      s += Gb[a + (int64_t)rp * (i + (int64_t)nk * b)] * Pp[(int64_t)a * Cp + i + (int64_t)nk * c];
    }
    s = wsum(s);
    if (lane == 0) Pkb[t] += s;
  }
}

// effective DRM value as the sketch kernels used it (see recover.hip)
__device__ __forceinline__ double drm_eff(double v, int prec) {
  if (prec == PSTT2_P_F64) return v;
  const float f = (float)v;
  if (prec == PSTT2_P_F16) return (double)(float)(_Float16)f;
  if (prec != PSTT2_P_BF16) return (double)f;
  uint32_t u = __float_as_uint(f);
  const uint32_t h = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return (double)__uint_as_float(h << 16);
}

// Pmbar(col, b) += sum_c Omega_m(col, c) Abar(b, c)
__global__ void k_pbar_from_abar(const double* __restrict__ om_tab, int L4, int64_t Cm, int rm, int ell, int prec,
                                 const double* __restrict__ Ab, double* __restrict__ Pb) {
  const int64_t tot = Cm * rm;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t col = t % Cm;
    const int b = (int)(t / Cm);
    double s = 0.0;
    for (int c = 0; c < ell; ++c) s += drm_eff(om_tab[col * L4 + c], prec) * Ab[b + (int64_t)rm * c];
    Pb[t] += s;
  }
}

// ---- thin-QR adjoints of every split's basis, three launches for all of them ----
// Problem k: basis Q (M x r), cotangent Qbar, sketch S whose pivoted columns piv
// give B = Q R.  (1) R = Q^T B and Mm = -Qbar^T Q, both from one read of a row
// slice, per slice on FP64 matrix cores (operands straight from memory: lane
// (g4, l16) holds rows 2 g4, 2 g4 + 1 of eight, column l16); (2) the slices' sums
// in slice order; (3) per row i: c = Qbar(i, :) + Q(i, :) copyltu(Mm), Bbar(i, :) R^T
// = c, Sbar(i, piv[j]) += Bbar(i, j).  Six launches a split and a division per
// back-substitution step took about 190 us for the four splits of n = 24^5; the
// three launches take 24.
constexpr int QA_ROWS = 512;   // rows per slice, 128 per wave
constexpr int QA_MAX = PSTT2_MAX_D;
struct QrAdjBatch {
  int n;
  const double *Q[QA_MAX], *Qb[QA_MAX], *S[QA_MAX];
  double* Sb[QA_MAX];
  const int* piv[QA_MAX];
  int64_t M[QA_MAX];
  int r[QA_MAX];
  int64_t slice0[QA_MAX + 1];   // first slice of each problem
  int64_t block0[QA_MAX + 1];   // first 256-row block of each problem
  double* part;                 // [slice][2][32 * 32]
  double* rm;                   // [problem][2][32 * 32]: R, then Mm
};

__device__ __forceinline__ int batch_of(const int64_t* first, int n, int64_t g) {
  int p = 0;
  while (p + 1 < n && first[p + 1] <= g) ++p;
  return p;
}

typedef double adj_d4 __attribute__((ext_vector_type(4)));

template <int RT>
__global__ __launch_bounds__(256) void k_qr_adj_prod(const QrAdjBatch B) {
  __shared__ double red[4][RT * RT * 256];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int p = batch_of(B.slice0, B.n, blockIdx.x);
  const int64_t M = B.M[p];
  const int r = B.r[p];
  const int64_t r0 = (blockIdx.x - B.slice0[p]) * QA_ROWS + 128 * w, r1 = r0 + 128 < M ? r0 + 128 : M;
  const double *q[RT], *qb[RT], *sp[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {   // columns past r read the last one; dropped below
    const int c = 16 * i + l16 < r ? 16 * i + l16 : r - 1;
    q[i] = B.Q[p] + c * M;
    qb[i] = B.Qb[p] + c * M;
    sp[i] = B.S[p] + B.piv[p][c] * M;
  }
  adj_d4 R[RT][RT], Mm[RT][RT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < RT; ++j) R[i][j] = Mm[i][j] = adj_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int64_t a = r0; a < r1; a += 8) {
    double x[RT][2], y[RT][2], z[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int64_t row = a + 2 * g4 + e;
        const bool in = row < r1;
        const int64_t rc = in ? row : r0;
        const double vx = q[i][rc], vy = qb[i][rc], vz = sp[i][rc];
        x[i][e] = in ? vx : 0.0;
        y[i][e] = in ? vy : 0.0;
        z[i][e] = in ? vz : 0.0;
      }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) {
          R[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][e], z[j][e], R[i][j], 0, 0, 0);
          Mm[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[i][e], x[j][e], Mm[i][j], 0, 0, 0);
        }
  }
  double* out = B.part + (int64_t)blockIdx.x * 2048;
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          red[w][(i * RT + j) * 256 + l16 * 16 + 4 * v + g4] = h == 0 ? R[i][j][v] : -Mm[i][j][v];
    __syncthreads();
    for (int o = t; o < r * r; o += 256) {
      const int a = o % r, b = o / r;
      const int e = ((a >> 4) * RT + (b >> 4)) * 256 + (b & 15) * 16 + (a & 15);
      out[h * 1024 + o] = red[0][e] + red[1][e] + red[2][e] + red[3][e];
    }
  }
}

__global__ __launch_bounds__(256) void k_qr_adj_sum(const QrAdjBatch B) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.y, r = B.r[p];
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= 2 * r * r) return;
  const int e = (o / (r * r)) * 1024 + o % (r * r);
  double s = 0.0;
  for (int64_t g = B.slice0[p] + lane; g < B.slice0[p + 1]; g += 64) s += B.part[g * 2048 + e];
  s = wsum(s);
  if (lane == 0) B.rm[(int64_t)p * 2048 + e] = s;
}

template <int RP>
__global__ __launch_bounds__(256) void k_qr_adj_rows(const QrAdjBatch B) {
  __shared__ double Rs[RP][RP + 1], Cs[RP][RP + 1], inv[RP];
  const int t = threadIdx.x;
  const int p = batch_of(B.block0, B.n, blockIdx.x);
  const int r = B.r[p];
  const int64_t M = B.M[p], i = (blockIdx.x - B.block0[p]) * 256 + t;
  const double *Q = B.Q[p], *Qb = B.Qb[p], *Rm = B.rm + (int64_t)p * 2048, *Mm = Rm + 1024;
  double q[RP], c[RP];
#pragma unroll
  for (int j = 0; j < RP; ++j) {
    const bool in = j < r && i < M;
    q[j] = in ? Q[j * M + i] : 0.0;
    c[j] = in ? Qb[j * M + i] : 0.0;
  }
  for (int o = t; o < RP * RP; o += 256) {
    const int a = o % RP, b = o / RP;
    const bool in = a < r && b < r;
    Rs[a][b] = in ? Rm[a + r * b] : 0.0;
    // copyltu: lower triangle (a >= b) kept, upper mirrored from the lower
    Cs[a][b] = in ? (a >= b ? Mm[a + r * b] : Mm[b + r * a]) : 0.0;
    if (a == b) inv[a] = in ? 1.0 / Rm[a + r * a] : 0.0;
  }
  __syncthreads();
  if (i >= M) return;
#pragma unroll
  for (int j = 0; j < RP; ++j)
#pragma unroll
    for (int l = 0; l < RP; ++l) c[j] += q[l] * Cs[l][j];
  // sum_{l >= j} R(j, l) x(l) = c(j), from the last j down
#pragma unroll
  for (int j = RP - 1; j >= 0; --j) {
#pragma unroll
    for (int l = j + 1; l < RP; ++l) c[j] -= Rs[j][l] * c[l];
    c[j] *= inv[j];
  }
#pragma unroll
  for (int j = 0; j < RP; ++j)
    if (j < r) B.Sb[p][B.piv[p][j] * M + i] += c[j];
}

// Sbar_{k+1}(row + Rk i, c) += Sbar_k(row, c) omega_{k+1}(i, c)   (adjoint of derive_left)
__global__ void k_derive_left_adj(const double* __restrict__ Sbk, double* __restrict__ Sbk1, int64_t Rk, int nk1,
                                  int ell, const double* __restrict__ om) {
  const int64_t Rk1 = Rk * nk1;
  const int64_t tot = Rk1 * ell;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rr = t % Rk1;
    const int c = (int)(t / Rk1);
    const int64_t row = rr % Rk;
    const int i = (int)(rr / Rk);
    Sbk1[t] += Sbk[(int64_t)c * Rk + row] * om[i * ell + c];
  }
}

// Tbar_{k-1}(i + nk col, a) += psi_k(i, a) Tbar_k(col, a)   (adjoint of derive_right; C x ell layouts)
__global__ void k_derive_right_adj(const double* __restrict__ Tbk, double* __restrict__ Tbp, int64_t Ck, int nk,
                                   int ell, const double* __restrict__ ps) {
  const int64_t Cp = Ck * nk;
  const int64_t tot = Cp * ell;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t cc = t % Cp;
    const int a = (int)(t / Cp);
    const int i = (int)(cc % nk);
    const int64_t col = cc / nk;
    Tbp[t] += ps[i * ell + a] * Tbk[(int64_t)a * Ck + col];
  }
}

// ---- B3: gx(row, col) = sum_c Ybar(row, c) Omega(col, c) + sum_a Psi(row, a) Tbar(col, a)
//                         [ + 2 (x - X~) for the fused loss ] [ + gx for ACC ] ----
// A product with inner dimension ell + ell (+ r for the -2 L Rt of the fused loss)
// on FP64 matrix cores: a wave owns 32 rows whose operands stay in registers for
// its whole share of the columns (KS steps of four), and forms 64-column tiles,
// columns on the M index, so a store covers 16 consecutive rows.  A null Yb or Tbt
// drops that term (a pass group of the independent scheme with only one side);
// ACC adds into gx (the later groups).  The column operands of a tile pass through
// LDS: loaded straight into registers they left one wave to a SIMD (98 us).  Bound
// by the matrix unit and the tiles' staging; x in and gx out alone would be 27 us.
// 24^5 FP64, ell = 20, r = 8: 60.5 us (2.1 TB/s); the vector version, one thread a
// row, took 93.  48^4 FP32, ell = 12, J^T alone: 29 -> 18 us.
struct AdjOutArgs {
  int64_t R, C;
  int ell, r, L4, prec;
  int n1, n2, n3;        // steps of the three terms (0: absent)
  const double* Yb;      // R x ell
  const double* psi;     // R x ell
  const double* L;       // R x r   (fused loss only)
  const double* om_tab;  // C x L4
  const double* Tbt;     // C x ell
  const double* Rt;      // r x C   (fused loss only)
  int gi, gj;            // row blocks of the launch, column shares
  int64_t row0;          // first row of the launch
};

constexpr int AO_ROWS = 128, AO_COLS = 64;

template <typename T, bool FUSED, bool ACC, int KS>
__global__ __launch_bounds__(256, 2) void k_adj_out(const AdjOutArgs A, const T* __restrict__ x, T* __restrict__ gx) {
  constexpr int LD = AO_COLS + 2;
  __shared__ double Co[4 * KS][LD];   // column operands of a tile, [inner index][column]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int64_t gi = blockIdx.x % A.gi, gj = blockIdx.x / A.gi;
  const int64_t row0 = A.row0 + gi * AO_ROWS + 32 * w;
  const int ks = A.n1 + A.n2 + A.n3;
  int64_t row[2];
  double ro[KS][2];   // row operands, zero past a term's length and past the matrix
#pragma unroll
  for (int t = 0; t < 2; ++t) row[t] = row0 + 16 * t + l16;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int c1 = 4 * s + g4, c2 = c1 - 4 * A.n1, c3 = c2 - 4 * A.n2;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      double v = 0.0;
      if (row[t] < A.R) {
        if (s < A.n1) {
          if (c1 < A.ell) v = A.Yb[c1 * A.R + row[t]];
        } else if (s < A.n1 + A.n2) {
          if (c2 < A.ell) v = drm_eff(A.psi[c2 * A.R + row[t]], A.prec);
        } else if (s < ks) {
          if (c3 < A.r) v = -2.0 * A.L[c3 * A.R + row[t]];
        }
      }
      ro[s][t] = v;
    }
  }
  const int64_t ntile = (A.C + AO_COLS - 1) / AO_COLS;
  for (int64_t tile = gj * ntile / A.gj; tile < (gj + 1) * ntile / A.gj; ++tile) {
    const int64_t cb = tile * AO_COLS;
    const int nc = (int)(A.C - cb < AO_COLS ? A.C - cb : AO_COLS);
    __syncthreads();   // the last tile's reads are done
    // Omega rows (their padding columns are zero), Tbar, Rt; zero past a term and past the matrix
    for (int e = tid; e < AO_COLS * 4 * A.n1; e += 256) {
      const int j = e / (4 * A.n1), c = e - j * 4 * A.n1;
      Co[c][j] = j < nc ? drm_eff(A.om_tab[(cb + j) * A.L4 + c], A.prec) : 0.0;
    }
    for (int e = tid; e < AO_COLS * 4 * A.n2; e += 256) {
      const int j = e % AO_COLS, c = e / AO_COLS;
      Co[4 * A.n1 + c][j] = j < nc && c < A.ell ? A.Tbt[(int64_t)c * A.C + cb + j] : 0.0;
    }
    for (int e = tid; e < AO_COLS * 4 * A.n3; e += 256) {
      const int j = e / (4 * A.n3), c = e - j * 4 * A.n3;
      Co[4 * (A.n1 + A.n2) + c][j] = j < nc && c < A.r ? A.Rt[c + (int64_t)A.r * (cb + j)] : 0.0;
    }
    __syncthreads();
    adj_d4 acc[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[u][t] = adj_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s < ks) {   // uniform
        double co[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) co[u] = Co[4 * s + g4][16 * u + l16];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(co[u], ro[s][t], acc[u][t], 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = 16 * u + 4 * v + g4;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if (j < nc && row[t] < A.R) {
            const int64_t f = (cb + j) * A.R + row[t];
            double g = acc[u][t][v];
            if constexpr (FUSED) g += 2.0 * (double)x[f];
            if constexpr (ACC) g += (double)gx[f];
            gx[f] = (T)g;
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
hipError_t adj_table(const double* in, int64_t rows, int cnt, int64_t si, int64_t sc, int L4, double* out,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_table, dim3(grid_for(rows * L4, 256)), dim3(256), 0, s, in, rows, cnt, si, sc, L4, out);
  return hipGetLastError();
}

hipError_t adj_transpose(const double* A, int64_t arows, int64_t acols, double* B, hipStream_t s) {
  hipLaunchKernelGGL(k_transpose, dim3(grid_for(arows * acols, 256)), dim3(256), 0, s, A, arows, acols, B);
  return hipGetLastError();
}

hipError_t adj_axpy(int64_t n, double alpha, const double* X, double* Y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpy, dim3(grid_for(n, 256)), dim3(256), 0, s, n, alpha, X, Y);
  return hipGetLastError();
}

hipError_t adj_ls(const double* G, const double* Gb, const double* Z, const double* A, int64_t p, int r, int ell,
                  double* Zb, double* Ab, hipStream_t s) {
  if (r <= 8) hipLaunchKernelGGL(k_ls_adjoint<8>, dim3(1), dim3(1024), 0, s, G, Gb, Z, A, p, r, ell, Zb, Ab);
  else if (r <= 16) hipLaunchKernelGGL(k_ls_adjoint<16>, dim3(1), dim3(1024), 0, s, G, Gb, Z, A, p, r, ell, Zb, Ab);
  else hipLaunchKernelGGL(k_ls_adjoint<32>, dim3(1), dim3(1024), 0, s, G, Gb, Z, A, p, r, ell, Zb, Ab);
  return hipGetLastError();
}

hipError_t adj_core_right(const double* Gb, const double* Pp, const double* Pk, int64_t Ck, int nk, int rp, int rk,
                          double* Ppb, double* Pkb, hipStream_t s) {
  hipLaunchKernelGGL(k_core_right_adj_prev, dim3(grid_for(Ck * nk * rp, 256)), dim3(256), 0, s, Gb, Pk, Ck, nk, rp, rk,
                     Ppb);
  hipLaunchKernelGGL(k_core_right_adj_next, dim3(grid_for(Ck * rk * 64, 256)), dim3(256), 0, s, Gb, Pp, Ck, nk, rp, rk,
                     Pkb);
  return hipGetLastError();
}

hipError_t adj_pbar(const double* om_tab, int L4, int64_t Cm, int rm, int ell, int prec, const double* Ab, double* Pb,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_pbar_from_abar, dim3(grid_for(Cm * rm, 256)), dim3(256), 0, s, om_tab, L4, Cm, rm, ell, prec,
                     Ab, Pb);
  return hipGetLastError();
}

hipError_t adj_qr_batch(int n, const double* const* S, const double* const* Q, const double* const* Qb,
                        const int64_t* M, const int* r, const int* const* piv, double* const* Sb, hipStream_t s) {
  QrAdjBatch B;
  std::memset(&B, 0, sizeof(B));
  B.n = n;
  int rmax = 1;
  for (int p = 0; p < n; ++p) {
    B.Q[p] = Q[p];
    B.Qb[p] = Qb[p];
    B.S[p] = S[p];
    B.Sb[p] = Sb[p];
    B.piv[p] = piv[p];
    B.M[p] = M[p];
    B.r[p] = r[p];
    rmax = std::max(rmax, r[p]);
    B.slice0[p + 1] = B.slice0[p] + (M[p] + QA_ROWS - 1) / QA_ROWS;
    B.block0[p + 1] = B.block0[p] + (M[p] + 255) / 256;
  }
  const int64_t slices = B.slice0[n];
  double* ws = nullptr;
  hipError_t e = ws_alloc((void**)&ws, sizeof(double) * 2048 * (slices + n), s);
  if (e != hipSuccess) return e;
  B.part = ws;
  B.rm = ws + 2048 * slices;
  if (rmax <= 16) hipLaunchKernelGGL(k_qr_adj_prod<1>, dim3((unsigned)slices), dim3(256), 0, s, B);
  else hipLaunchKernelGGL(k_qr_adj_prod<2>, dim3((unsigned)slices), dim3(256), 0, s, B);
  hipLaunchKernelGGL(k_qr_adj_sum, dim3((unsigned)((2 * rmax * rmax + 3) / 4), (unsigned)n), dim3(256), 0, s, B);
  const dim3 g((unsigned)B.block0[n]), b(256);
  if (rmax <= 8) hipLaunchKernelGGL(k_qr_adj_rows<8>, g, b, 0, s, B);
  else if (rmax <= 16) hipLaunchKernelGGL(k_qr_adj_rows<16>, g, b, 0, s, B);
  else hipLaunchKernelGGL(k_qr_adj_rows<32>, g, b, 0, s, B);
  e = hipGetLastError();
  ws_free(ws, s);
  return e;
}

__global__ void k_zero(double* __restrict__ p, int64_t n) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) p[t] = 0.0;
}

hipError_t adj_zero(double* p, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t adj_derive_left(const double* Sbk, double* Sbk1, int64_t Rk, int nk1, int ell, const double* om,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_derive_left_adj, dim3(grid_for(Rk * nk1 * ell, 256)), dim3(256), 0, s, Sbk, Sbk1, Rk, nk1, ell,
                     om);
  return hipGetLastError();
}

hipError_t adj_derive_right(const double* Tbk, double* Tbp, int64_t Ck, int nk, int ell, const double* ps,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_derive_right_adj, dim3(grid_for(Ck * nk * ell, 256)), dim3(256), 0, s, Tbk, Tbp, Ck, nk, ell,
                     ps);
  return hipGetLastError();
}

template <int KS>
static void launch_adj_out(int dtype, bool fused, bool acc, const AdjOutArgs& A, const void* x, void* gx,
                           hipStream_t s) {
  const dim3 grid((unsigned)((int64_t)A.gi * A.gj)), block(256);
  if (dtype == PSTT2_F64) {
    if (fused)
      hipLaunchKernelGGL((k_adj_out<double, true, false, KS>), grid, block, 0, s, A, (const double*)x, (double*)gx);
    else if (acc)
      hipLaunchKernelGGL((k_adj_out<double, false, true, KS>), grid, block, 0, s, A, (const double*)x, (double*)gx);
    else
      hipLaunchKernelGGL((k_adj_out<double, false, false, KS>), grid, block, 0, s, A, (const double*)x, (double*)gx);
  } else {
    if (fused)
      hipLaunchKernelGGL((k_adj_out<float, true, false, KS>), grid, block, 0, s, A, (const float*)x, (float*)gx);
    else if (acc)
      hipLaunchKernelGGL((k_adj_out<float, false, true, KS>), grid, block, 0, s, A, (const float*)x, (float*)gx);
    else
      hipLaunchKernelGGL((k_adj_out<float, false, false, KS>), grid, block, 0, s, A, (const float*)x, (float*)gx);
  }
}

hipError_t adj_out(int dtype, const SketchArgs& g, int prec, const double* Yb, const double* Tbt, const double* L,
                   const double* Rt, int r, const void* x, void* gx, bool acc, hipStream_t s) {
  const bool fused = L != nullptr;
  if (fused && acc) return hipErrorInvalidValue;   // the loss term enters once, in the first group
  if (g.ell > PSTT2_MAX_ELL || r > PSTT2_MAX_ELL) return hipErrorInvalidValue;
  AdjOutArgs A;
  std::memset(&A, 0, sizeof(A));
  A.R = g.R;
  A.C = g.C;
  A.ell = g.ell;
  A.r = r;
  A.L4 = g.L4;
  A.prec = prec;
  A.n1 = Yb ? (g.ell + 3) / 4 : 0;
  A.n2 = Tbt ? (g.ell + 3) / 4 : 0;
  A.n3 = fused ? (r + 3) / 4 : 0;
  A.Yb = Yb;
  A.Tbt = Tbt;
  A.om_tab = g.om_tab;
  A.L = L;
  A.Rt = Rt;
  double* psi = nullptr;
  hipError_t e = hipSuccess;
  if (Tbt) {   // the left DRM of this group's factors, R x ell
    KRChain ch;
    std::memset(&ch, 0, sizeof(ch));
    for (int q = 0; q < g.m; ++q) {
      ch.n[ch.cnt] = g.n[q];
      ch.off[ch.cnt++] = g.psi_off[q];
    }
    e = ws_alloc((void**)&psi, sizeof(double) * g.R * g.ell, s);
    if (e == hipSuccess) e = kr_table(g.fac, ch, g.R, g.ell, psi, s);
    if (e != hipSuccess) return e;
  }
  A.psi = psi;
  const int64_t blocks = (g.R + AO_ROWS - 1) / AO_ROWS, ntile = (g.C + AO_COLS - 1) / AO_COLS;
  constexpr int64_t kMaxBlocks = 1 << 22;   // a launch has less than 2^32 threads
  const int ks = A.n1 + A.n2 + A.n3;
  for (int64_t b0 = 0; b0 < blocks && e == hipSuccess; b0 += kMaxBlocks) {
    A.row0 = b0 * AO_ROWS;
    A.gi = (int)std::min(blocks - b0, kMaxBlocks);
    A.gj = (int)std::max<int64_t>(1, std::min<int64_t>(ntile, (2048 + A.gi - 1) / A.gi));
    if (ks <= 6) launch_adj_out<6>(dtype, fused, acc, A, x, gx, s);
    else if (ks <= 12) launch_adj_out<12>(dtype, fused, acc, A, x, gx, s);
    else if (ks <= 18) launch_adj_out<18>(dtype, fused, acc, A, x, gx, s);
    else launch_adj_out<24>(dtype, fused, acc, A, x, gx, s);
    e = hipGetLastError();
  }
  ws_free(psi, s);
  return e;
}

}  // namespace pstt2
