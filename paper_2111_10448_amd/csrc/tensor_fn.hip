// Tensors given by a formula of their indices (the streaming setting of
// Section 4.2, where each sub-tensor comes from a function of its indices and
// is never stored as a whole).  The Hilbert tensor of Section 4.3 / Table 1,
//     X(i_1, ..., i_d) = 1 / (1 - d + i_1 + ... + i_d),   1 <= i_q <= n_q,
// depends on the indices only through their sum.  On the split X_m (rows =
// modes 1..m, columns = modes m+1..d) that sum is a row part plus a column
// part, so X(row, col) = rec[row_t[row] + col_t[col]] with
//     row_t[row] = 1 + sum of the row's 0-based mode indices,
//     col_t[col] = sum of the column's 0-based mode indices,
//     rec[k]     = 1 / k (FP64, correctly rounded).
// The sketch and error kernels read these three small tables instead of X.
//
// The Gaussian-bump tensor of Section 4.4,
//     X(i) = sum_j exp(-gamma sum_q (x_q - c_{j,q})^2),   x_q = 2 i_q / n_q - 1,
// is a sum of products of one factor per mode, e_q(i_q, j) =
// exp(-gamma (x_q - c_{j,q})^2).  On X_m that is X(row, col) = sum_j
// a(row, j) b(col, j) with a = e_1(i_1, j) h(row / n_1, j), h the product of
// the factors of modes 2..m and b that of modes m+1..d.  The three tables are
// small (N (n_1 + R_m / n_1 + C_m) doubles); gauss_columns evaluates chunks of
// whole columns of X_m from them into a workspace that the memory kernels
// stream, at 2N FP64 flops per entry; gauss_error compares every entry with a
// train's without storing any; and FP64 contexts sketch the tensor from the
// factors' moments (gauss_moments and the two kernels after it).
#include <hip/hip_runtime.h>

#include "internal.h"

namespace pstt2 {

namespace {

// 0-based mode indices of a flat index over modes q0 .. q1-1 (first fastest), summed
__device__ __forceinline__ int32_t digit_sum(int64_t f, const int64_t* n, int q0, int q1) {
  int32_t s = 0;
  for (int q = q0; q < q1; ++q) {
    s += (int32_t)(f % n[q]);
    f /= n[q];
  }
  return s;
}

struct Modes {
  int64_t n[PSTT2_MAX_D];
};

__global__ void k_hilbert_tables(const Modes M, int d, int m, int64_t R, int64_t C, int64_t K,
                                 double* __restrict__ rec, int32_t* __restrict__ row_t,
                                 int32_t* __restrict__ col_t) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t i = t0; i < R; i += stride) row_t[i] = 1 + digit_sum(i, M.n, 0, m);
  for (int64_t i = t0; i < C; i += stride) col_t[i] = digit_sum(i, M.n, m, d);
  for (int64_t k = t0; k < K; k += stride) rec[k] = k == 0 ? 0.0 : 1.0 / (double)k;
}

// out[j * cnt + f] = prod over modes q0..q1-1 of exp(-gamma (x_q - c_{j,q})^2), f a flat
// index over those modes (first fastest), x_q = 2 (i_q + 1) / n_q - 1 (0-based i_q)
__global__ void k_gauss_table(const Modes M, int q0, int q1, int64_t cnt, int64_t stride, const double* __restrict__ ctr,
                              int d, int nterms, double gamma, double* __restrict__ out) {
  const int64_t tot = cnt * nterms;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(t / cnt);
    int64_t f = t % cnt;
    double v = 1.0;
    for (int q = q0; q < q1; ++q) {
      const int64_t i = f % M.n[q];
      f /= M.n[q];
      const double x = 2.0 * (double)(i + 1) / (double)M.n[q] - 1.0;
      const double dl = x - ctr[(int64_t)j * d + q];
      v *= exp(-gamma * (dl * dl));
    }
    out[(int64_t)j * stride + t % cnt] = v;
  }
}

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kGaussRows = 256;   // rows of X_m per workgroup of k_gauss_tiles
constexpr int kGaussTile = 64;    // columns per step

// Tiles of X_m = sum_j a(:, j) b(:, j)^T on FP64 matrix cores: a product with the
// bumps as its inner dimension.  A workgroup owns 256 rows and a share of the
// 64-column tiles; a wave holds 64 x 64 entries in 16 accumulator tiles, so a
// step of four bumps costs 16 matrix instructions (1024 cycles) for twelve
// loads of cached table entries, requested one step ahead.  The columns are the
// M index and the rows the N index: element v of a tile is (row l16, column
// 4 v + g4), so a store instruction covers 16 consecutive rows.
// ERR: nothing is stored.  The sum of x^2 is taken from the tile, then -L Rt is
// added on the matrix cores (RK more inner steps) and the sum of squares taken
// again: sum (x - x~)^2 by entrywise differences.
// Bound by the FP64 matrix cores (2 nterms flops per entry).  At n = 960^3 with
// 100 bumps the vector version (39 TFLOP/s) took 4.5 ms into workspace chunks of
// 4 GiB, and the error pass then 1.4 ms to read them back; the chunks now take
// 3.9 ms and the error pass, at rank 12, 3.7 ms in all (53 TFLOP/s).
struct GaussErr {
  const double* L;    // R x r
  const double* Rp;   // RK x C, zero past r
  int r, RK;
  double* part;       // (sum (x - x~)^2, sum x^2) per workgroup
};

template <bool ERR, typename T>
__global__ __launch_bounds__(256, 2) void k_gauss_tiles(const GaussTabs g, int64_t c0, int64_t nc, T* __restrict__ W,
                                                        const GaussErr er, int64_t gi0, int gi_count, int gj_count) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int64_t gi = gi0 + blockIdx.x % gi_count, gj = blockIdx.x / gi_count;
  const int64_t row0 = gi * kGaussRows + 64 * w;
  const int64_t ntile = (nc + kGaussTile - 1) / kGaussTile;
  const int nt = g.nterms;
  // rows past the matrix read its last row, columns past it its last column; both are dropped at the end
  const double *pe[4], *ph[4];
  int64_t row[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    row[t] = row0 + 16 * t + l16;
    const int64_t rr = row[t] < g.R ? row[t] : g.R - 1;
    pe[t] = g.e1 + rr % g.n1;
    ph[t] = g.ahi + rr / g.n1;
  }
  double e2 = 0.0, x2 = 0.0;
  for (int64_t tile = gj * ntile / gj_count; tile < (gj + 1) * ntile / gj_count; ++tile) {
    const int64_t cc = c0 + tile * kGaussTile;
    const double* pb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t c = cc + 16 * t + l16;
      pb[t] = g.bc + (c < g.C ? c : g.C - 1);
    }
    d4 acc[4][4];   // [column tile][row tile]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
    // table offsets of this lane's bump; a lane whose next bump would be past the
    // last one stays (its operand is zeroed)
    int64_t oe = 0, oh = 0, ob = 0;
    {
      const int64_t j = g4 < nt ? g4 : nt - 1;
      oe = j * g.n1;
      oh = j * g.rhi;
      ob = j * g.bstride;
    }
    double ve[4], vh[4], vb[4];
    auto load = [&]() {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        ve[t] = pe[t][oe];
        vh[t] = ph[t][oh];
        vb[t] = pb[t][ob];
      }
    };
    load();
    for (int j0 = 0; j0 < nt; j0 += 4) {
      double a[4], b[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[t] = ve[t] * vh[t];
        b[t] = j0 + g4 < nt ? vb[t] : 0.0;
      }
      const bool more = j0 + 4 + g4 < nt;
      oe += more ? 4 * g.n1 : 0;
      oh += more ? 4 * g.rhi : 0;
      ob += more ? 4 * g.bstride : 0;
      load();
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) acc[ct][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[ct], a[rt], acc[ct][rt], 0, 0, 0);
    }
    if constexpr (ERR) {
      const bool whole = row0 + 64 <= g.R && cc + kGaussTile <= c0 + nc;   // uniform
      auto squares = [&]() {
        double s = 0.0;
        if (whole) {
#pragma unroll
          for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int rt = 0; rt < 4; ++rt)
#pragma unroll
              for (int v = 0; v < 4; ++v) s += acc[ct][rt][v] * acc[ct][rt][v];
          return s;
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const bool cok = cc + 16 * ct + 4 * v + g4 < c0 + nc;
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) {
              const double x = cok && row[rt] < g.R ? acc[ct][rt][v] : 0.0;
              s += x * x;
            }
          }
        return s;
      };
      x2 += squares();
      for (int b0 = 0; b0 < er.RK; b0 += 4) {
        const int b = b0 + g4;
        double lv[4], rv[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int64_t rr = row[t] < g.R ? row[t] : g.R - 1;
          lv[t] = b < er.r ? er.L[(int64_t)b * g.R + rr] : 0.0;
          rv[t] = -er.Rp[(pb[t] - g.bc) * er.RK + b];
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int rt = 0; rt < 4; ++rt)
            acc[ct][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(rv[ct], lv[rt], acc[ct][rt], 0, 0, 0);
      }
      e2 += squares();
    } else {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t c = cc + 16 * ct + 4 * v + g4;
          if (c < c0 + nc) {
#pragma unroll
            for (int rt = 0; rt < 4; ++rt)
              if (row[rt] < g.R) W[(c - c0) * g.R + row[rt]] = (T)acc[ct][rt][v];
          }
        }
    }
  }
  if constexpr (ERR) {
    __shared__ double red[2][4];
    for (int o = 32; o > 0; o >>= 1) {
      e2 += __shfl_xor(e2, o);
      x2 += __shfl_xor(x2, o);
    }
    if (lane == 0) {
      red[0][w] = e2;
      red[1][w] = x2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double* part = er.part + 2 * (gi + (g.R + kGaussRows - 1) / kGaussRows * gj);
      part[0] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
      part[1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
  }
}

// Row blocks and column shares: about 10000 workgroups, so that the last of the
// (two per compute unit) rounds they run in is a small part of the whole.
void gauss_grid(const GaussTabs& g, int64_t nc, int64_t* gi, int* gj) {
  *gi = (g.R + kGaussRows - 1) / kGaussRows;
  const int64_t ntile = (nc + kGaussTile - 1) / kGaussTile;
  *gj = (int)std::max<int64_t>(1, std::min<int64_t>(ntile, (10240 + *gi - 1) / *gi));
}

template <bool ERR, typename T>
hipError_t launch_tiles(const GaussTabs& g, int64_t c0, int64_t nc, T* W, const GaussErr& er, hipStream_t s) {
  constexpr int64_t kMaxBlocks = 1 << 22;   // a launch has less than 2^32 threads
  int64_t gi = 1;
  int gj = 1;
  gauss_grid(g, nc, &gi, &gj);
  for (int64_t b0 = 0; b0 < gi; b0 += kMaxBlocks) {
    const int n = (int)std::min(gi - b0, kMaxBlocks);
    hipLaunchKernelGGL((k_gauss_tiles<ERR, T>), dim3((unsigned)((int64_t)n * gj)), dim3(256), 0, s, g, c0, nc, W, er, b0,
                       n, gj);
  }
  return hipGetLastError();
}

// ---- sketches of the Gaussian bumps without their entries ----
// X_m = sum_j a_j b_j^T, so X_m Omega = sum_j a_j (b_j^T Omega) and Psi^T X_m =
// sum_j (a_j^T Psi)^T b_j^T: the sketches need the bumps' moments, nterms x ell
// numbers on either side.  Psi is a Khatri-Rao product and a_j a product of one
// factor per mode, so a_j^T Psi is a product over modes of length-n_q dots.  All
// in FP64; every term of the sums is the one that the entries would give, added
// in another order.  At n = 960^3, 100 bumps, ell = 32 this is 0.012 TFLOP of
// work in place of 0.29 (evaluation and sketch), bound by writing Y_R: the call
// went from 7.1 to 0.30 ms (0.22 ms of it k_gauss_y).
//
// moments: workgroup j < nterms: mpsi[32 j + a] = a_j^T Psi(:, a); the others:
// mom[32 j + c] = sum over the columns [c0, c0 + nc) of b_j(col) Omega(col, c).
// 32 groups of 32 threads (one sketch column each), summed in group order.
__global__ __launch_bounds__(1024) void k_gauss_moments(const GaussTabs g, const SketchArgs A, const Modes M, int d,
                                                        double gamma, int64_t c0, int64_t nc,
                                                        double* __restrict__ mpsi, double* __restrict__ mom) {
  __shared__ double red[32][33];
  const int c = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int ell = A.ell;
  const int j = blockIdx.x < (unsigned)g.nterms ? blockIdx.x : blockIdx.x - g.nterms;
  const int cl = c < ell ? c : 0;
  auto total = [&](double v) {
    __syncthreads();
    red[grp][c] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 32; ++k) s += red[k][c];
    return s;
  };
  if (blockIdx.x < (unsigned)g.nterms) {
    double prod = 1.0;
    for (int q = 1; q <= A.m; ++q) {
      const int64_t nq = M.n[q - 1];
      const double* f = A.fac + A.psi_off[q - 1] + cl;
      // the tables hold mode 1's factor, and mode 2's where it is the last row mode
      const double* tab = q == 1 ? g.e1 + (int64_t)j * g.n1 : (q == 2 && A.m == 2 ? g.ahi + (int64_t)j * g.rhi : nullptr);
      const double ctr = g.centers[(int64_t)j * d + q - 1];
      double s = 0.0;
#pragma unroll 4
      for (int64_t i = grp; i < nq; i += 32) {
        double e;
        if (tab) {
          e = tab[i];
        } else {
          const double dl = 2.0 * (double)(i + 1) / (double)nq - 1.0 - ctr;
          e = exp(-gamma * (dl * dl));
        }
        s += e * f[i * ell];
      }
      prod *= total(s);
    }
    if (grp == 0) mpsi[32 * j + c] = c < ell ? prod : 0.0;
  } else {
    const double* b = g.bc + (int64_t)j * g.bstride + c0;
    const double* om = A.om_tab + c0 * A.L4 + cl;
    double s = 0.0;
#pragma unroll 4
    for (int64_t i = grp; i < nc; i += 32) s += b[i] * om[i * A.L4];
    s = total(s);
    if (grp == 0) mom[32 * j + c] = c < ell ? s : 0.0;
  }
}

// Y(row, c) = [Y(row, c)] + sum_j a(row, j) mom(j, c): 256 rows per workgroup, a wave
// 64 rows x 16 CT sketch columns on the matrix cores, four bumps per step.
template <int CT>
__global__ __launch_bounds__(256) void k_gauss_y(const GaussTabs g, const double* __restrict__ mom, int ell, bool store,
                                                 double* __restrict__ Y, int* flag) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int64_t row0 = blockIdx.x * (int64_t)256 + 64 * w;
  const double *pe[4], *ph[4];
  int64_t row[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    row[t] = row0 + 16 * t + l16;
    const int64_t rr = row[t] < g.R ? row[t] : g.R - 1;
    pe[t] = g.e1 + rr % g.n1;
    ph[t] = g.ahi + rr / g.n1;
  }
  d4 acc[CT][4];
#pragma unroll
  for (int a = 0; a < CT; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int j0 = 0; j0 < g.nterms; j0 += 4) {
    const int j = j0 + g4;
    const bool in = j < g.nterms;
    const int64_t jj = in ? j : g.nterms - 1;
    double a[4], m[CT];
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = pe[t][jj * g.n1] * ph[t][jj * g.rhi];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const double v = mom[32 * jj + 16 * ct + l16];
      m[ct] = in ? v : 0.0;
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[ct][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[ct], a[t], acc[ct][t], 0, 0, 0);
  }
  bool bad = false;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * ct + 4 * v + g4;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (c < ell && row[t] < g.R) {
          double* y = Y + (int64_t)c * g.R + row[t];
          const double s = (store ? 0.0 : *y) + acc[ct][t][v];
          *y = s;
          bad = bad || !isfinite(s);
        }
    }
  if (bad) atomicOr(flag, 1);
}

// T(a, col) += sum_j b_j(col) mpsi(j, a) for the columns [c0, c0 + nc)
__global__ __launch_bounds__(256) void k_gauss_t(const GaussTabs g, const double* __restrict__ mpsi, int64_t c0,
                                                 int64_t nc, double* __restrict__ Tt, int* flag) {
  const int a = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < nc; i += (int64_t)gridDim.x * 256) {
    const double* b = g.bc + c0 + i;
    double s = 0.0;
#pragma unroll 8
    for (int j = 0; j < g.nterms; ++j) s += b[(int64_t)j * g.bstride] * mpsi[32 * j + a];
    double* t = Tt + (int64_t)a * g.C + c0 + i;
    s += *t;
    *t = s;
    if (!isfinite(s)) atomicOr(flag, 1);
  }
}

// W(row, c) = rec[row_t[row] + col_t[c0 + c]] for the columns [c0, c0 + nc) of X_m
template <typename T>
__global__ void k_hilbert_cols(const double* __restrict__ rec, const int32_t* __restrict__ row_t,
                               const int32_t* __restrict__ col_t, int64_t R, int64_t c0, int64_t nc,
                               T* __restrict__ W) {
  const int64_t tot = R * nc;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x)
    W[t] = (T)rec[row_t[t % R] + col_t[c0 + t / R]];
}

unsigned grid1(int64_t work) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, 4096));
}

}  // namespace

int64_t gauss_table_doubles(const int64_t* n, int d, int m, int nterms) {
  int64_t R = 1, C = 1;
  for (int q = 0; q < m; ++q) R *= n[q];
  for (int q = m; q < d; ++q) C *= n[q];
  return (int64_t)nterms * (d + n[0] + R / n[0] + C + kGaussPad);
}

hipError_t gauss_tables(const int64_t* n, int d, int m, const double* centers_host, int nterms, double gamma,
                        double* buf, GaussTabs* out, hipStream_t s) {
  if (fault_take()) return hipErrorLaunchFailure;
  Modes M;
  for (int q = 0; q < PSTT2_MAX_D; ++q) M.n[q] = q < d ? n[q] : 1;
  int64_t R = 1, C = 1;
  for (int q = 0; q < m; ++q) R *= n[q];
  for (int q = m; q < d; ++q) C *= n[q];
  GaussTabs g;
  g.nterms = nterms;
  g.n1 = n[0];
  g.rhi = R / n[0];
  g.R = R;
  g.C = C;
  g.bstride = C + kGaussPad;
  double* ctr = buf;
  double* e1 = ctr + (int64_t)nterms * d;
  double* ahi = e1 + (int64_t)nterms * g.n1;
  double* bc = ahi + (int64_t)nterms * g.rhi;
  g.centers = ctr;
  g.e1 = e1;
  g.ahi = ahi;
  g.bc = bc;
  // the centers are read by the kernels below only; copy them and wait, so the
  // caller's host array may go as soon as this returns
  hipError_t e = hipMemcpyAsync(ctr, centers_host, sizeof(double) * nterms * d, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gauss_table, dim3(grid1(g.n1 * nterms)), dim3(256), 0, s, M, 0, 1, g.n1, g.n1, ctr, d,
                     nterms, gamma, e1);
  hipLaunchKernelGGL(k_gauss_table, dim3(grid1(g.rhi * nterms)), dim3(256), 0, s, M, 1, m, g.rhi, g.rhi, ctr, d,
                     nterms, gamma, ahi);
  hipLaunchKernelGGL(k_gauss_table, dim3(grid1(C * nterms)), dim3(256), 0, s, M, m, d, C, g.bstride, ctr, d, nterms,
                     gamma, bc);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  *out = g;
  return hipStreamSynchronize(s);
}

int64_t gauss_chunk_cols(const GaussTabs& g, int elem_bytes) {
  int64_t by_bytes = std::max<int64_t>(1, PSTT2_GAUSS_CHUNK_BYTES / (g.R * elem_bytes));
  if (by_bytes > kGaussTile) by_bytes -= by_bytes % kGaussTile;   // whole column tiles
  return std::min(by_bytes, g.C);
}

hipError_t gauss_columns(const GaussTabs& g, int64_t c0, int64_t nc, int dtype, void* W, hipStream_t s) {
  if (nc <= 0) return hipSuccess;
  if (fault_take()) return hipErrorLaunchFailure;
  const GaussErr none = {};
  if (dtype == PSTT2_F64) return launch_tiles<false>(g, c0, nc, (double*)W, none, s);
  return launch_tiles<false>(g, c0, nc, (float*)W, none, s);
}

hipError_t gauss_moments(const GaussTabs& g, const SketchArgs& a, const int64_t* n, double gamma, int64_t c0,
                         int64_t nc, double* mom, hipStream_t s) {
  if (fault_take()) return hipErrorLaunchFailure;
  Modes M;
  for (int q = 0; q < PSTT2_MAX_D; ++q) M.n[q] = q < a.d ? n[q] : 1;
  hipLaunchKernelGGL(k_gauss_moments, dim3(2 * (unsigned)g.nterms), dim3(1024), 0, s, g, a, M, a.d, gamma, c0, nc, mom,
                     mom + 32 * (int64_t)g.nterms);
  return hipGetLastError();
}

hipError_t gauss_sketch_y(const GaussTabs& g, const double* mom, int ell, bool store, double* Y, int* flag,
                          hipStream_t s) {
  if (fault_take()) return hipErrorLaunchFailure;
  const dim3 grid((unsigned)((g.R + 255) / 256)), b(256);
  const double* m = mom + 32 * (int64_t)g.nterms;
  if (ell <= 16) hipLaunchKernelGGL(k_gauss_y<1>, grid, b, 0, s, g, m, ell, store, Y, flag);
  else hipLaunchKernelGGL(k_gauss_y<2>, grid, b, 0, s, g, m, ell, store, Y, flag);
  return hipGetLastError();
}

hipError_t gauss_sketch_t(const GaussTabs& g, const double* mom, int ell, int64_t c0, int64_t nc, double* Tt, int* flag,
                          hipStream_t s) {
  if (fault_take()) return hipErrorLaunchFailure;
  const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>((nc + 255) / 256, 4096)), (unsigned)ell);
  hipLaunchKernelGGL(k_gauss_t, grid, dim3(256), 0, s, g, mom, c0, nc, Tt, flag);
  return hipGetLastError();
}

int64_t gauss_error_parts(const GaussTabs& g) {
  int64_t gi = 1;
  int gj = 1;
  gauss_grid(g, g.C, &gi, &gj);
  return gi * gj;
}

hipError_t gauss_error(const GaussTabs& g, const double* L, const double* Rp, int r, int RK, double* part,
                       hipStream_t s) {
  if (fault_take()) return hipErrorLaunchFailure;
  return launch_tiles<true>(g, 0, g.C, (double*)nullptr, GaussErr{L, Rp, r, RK, part}, s);
}

hipError_t hilbert_columns(const double* rec, const int32_t* row_t, const int32_t* col_t, int64_t R, int64_t c0,
                           int64_t nc, int dtype, void* W, hipStream_t s) {
  if (nc <= 0) return hipSuccess;
  if (fault_take()) return hipErrorLaunchFailure;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((R * nc + 255) / 256, 65536));
  if (dtype == PSTT2_F64)
    hipLaunchKernelGGL(k_hilbert_cols<double>, dim3(g), dim3(256), 0, s, rec, row_t, col_t, R, c0, nc, (double*)W);
  else
    hipLaunchKernelGGL(k_hilbert_cols<float>, dim3(g), dim3(256), 0, s, rec, row_t, col_t, R, c0, nc, (float*)W);
  return hipGetLastError();
}

hipError_t hilbert_tables(const int64_t* n, int d, int m, int64_t R, int64_t C, double* rec, int32_t* row_t,
                          int32_t* col_t, hipStream_t s) {
  Modes M;
  for (int q = 0; q < PSTT2_MAX_D; ++q) M.n[q] = q < d ? n[q] : 1;
  const int64_t K = hilbert_rec_len(n, d);
  const int64_t work = std::max(std::max(R, C), K);
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, 4096));
  hipLaunchKernelGGL(k_hilbert_tables, dim3(g), dim3(256), 0, s, M, d, m, R, C, K, rec, row_t, col_t);
  return hipGetLastError();
}

}  // namespace pstt2
