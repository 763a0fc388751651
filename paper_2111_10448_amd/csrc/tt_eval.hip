// Evaluation of a tensor train against a dense tensor (Section 2.2 entry
// formula; relative Frobenius error of equation "FrobeniusNorm").
//
// The train is split at mode m: the left interface L (R_m x r_m) holds the
// products G_1(i_1) ... G_m(i_m) for every row of X_m and the right interface
// Rt (r_m x C_m) the products G_{m+1}(i_{m+1}) ... G_d(i_d) for every column, so
// that X~_m = L Rt.  tt_error streams X once: lanes run along rows with 8- or
// 16-byte loads (each column of X_m is contiguous), every lane keeps its rows
// of L in registers, and the column's Rt(:, col) is wave-uniform (scalar
// loads).  Squared differences are summed in FP64, never through
// ||X||^2 - 2<X, X~> + ||X~||^2, which cancels.
#include <algorithm>
#include <mutex>

#include "internal.h"

namespace pstt2 {

static unsigned grid_for(int64_t n, int bs) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + bs - 1) / bs, 8192));
}

// One level of both interfaces in one launch (the two chains are independent):
//   left   L_k(row + R_{k-1} i, b) = sum_a L_{k-1}(row, a) G_k(a, i, b),
//          workgroups [0, gl): one thread per row of L_k, its rp entries of
//          L_{k-1} read once and kept in registers for all rk outputs;
//   right  Rt_k(a, i + n_k col) = sum_b G_k(a, i, b) Rt_{k+1}(b, col), Rt_{k+1}
//          r_k x C_k, workgroups [gl, gl + gr): one thread per entry.  The last
//          level is written with ldr >= r rows per column, zero past r (the
//          streaming kernels read a column's entries as one run of that length).
// Latency bound (a few microseconds a level at the sizes of a middle split): the
// chains' levels share launches, and the register slots of the left part are
// rounded up from the rank, so its loop has no guard per entry.  At R = 20592,
// r = 8 a left level took 10.8 us with 32 guarded slots, 5 launches for d = 8.
struct IfaceLevel {
  const double *Lp, *Gl;
  double* L;
  int64_t Rp;
  int rpl, nl, rkl;
  unsigned gl;
  const double *Gr, *Rn;
  double* Rt;
  int64_t Ck;
  int rpr, nr, rkr, ldr;
  unsigned gr;
};

template <int RP>
__global__ __launch_bounds__(256) void k_ifaces(const IfaceLevel A) {
  constexpr int LO = RP > 16 ? RP - 8 : RP - 4;   // the ranks of these slots are above it
  if (blockIdx.x < A.gl) {
    const int64_t Rk = A.Rp * A.nl;
    const int rp = A.rpl;
    for (int64_t rr = blockIdx.x * (int64_t)256 + threadIdx.x; rr < Rk; rr += (int64_t)A.gl * 256) {
      const int i = (int)(rr / A.Rp);
      const int64_t row = rr - A.Rp * i;
      double lp[RP];
#pragma unroll
      for (int a = 0; a < RP; ++a) lp[a] = a < rp ? A.Lp[(int64_t)a * A.Rp + row] : 0.0;
      for (int b = 0; b < A.rkl; ++b) {
        const double* g = A.Gl + (int64_t)rp * (i + (int64_t)A.nl * b);
        double s = 0.0;
#pragma unroll
        for (int a = 0; a < RP; ++a) {
          const double gv = g[a < LO || a < rp ? a : 0];   // a finite product with lp = 0 past rp
          s += lp[a] * (a < LO || a < rp ? gv : 0.0);
        }
        A.L[rr + Rk * b] = s;
      }
    }
    return;
  }
  const int64_t Cp = A.Ck * A.nr;
  const int64_t tot = (int64_t)A.ldr * Cp;
  for (int64_t t = (blockIdx.x - A.gl) * (int64_t)256 + threadIdx.x; t < tot; t += (int64_t)A.gr * 256) {
    const int64_t cc = t / A.ldr;
    const int a = (int)(t - cc * A.ldr);
    const int64_t col = cc / A.nr;
    const int i = (int)(cc - col * A.nr);
    double s = 0.0;
    if (a < A.rpr)
      for (int b = 0; b < A.rkr; ++b)
        s += A.Gr[a + (int64_t)A.rpr * (i + (int64_t)A.nr * b)] * A.Rn[b + (int64_t)A.rkr * col];
    A.Rt[t] = s;
  }
}

static void launch_ifaces(const IfaceLevel& A, hipStream_t s) {
  const dim3 g(A.gl + A.gr), b(256);
  const int rp = A.gl ? A.rpl : 1;
  if (rp <= 4) hipLaunchKernelGGL(k_ifaces<4>, g, b, 0, s, A);
  else if (rp <= 8) hipLaunchKernelGGL(k_ifaces<8>, g, b, 0, s, A);
  else if (rp <= 12) hipLaunchKernelGGL(k_ifaces<12>, g, b, 0, s, A);
  else if (rp <= 16) hipLaunchKernelGGL(k_ifaces<16>, g, b, 0, s, A);
  else if (rp <= 24) hipLaunchKernelGGL(k_ifaces<24>, g, b, 0, s, A);
  else hipLaunchKernelGGL(k_ifaces<32>, g, b, 0, s, A);
}

// Rt (r x C, column-major) -> Rp (RK x C) with zero rows r..RK-1
__global__ void k_pad_rt(const double* __restrict__ Rt, int r, int RK, int64_t C, double* __restrict__ Rp) {
  const int64_t tot = (int64_t)RK * C;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(t % RK);
    Rp[t] = k < r ? Rt[(t / RK) * r + k] : 0.0;
  }
}

// Doubles of every intermediate interface level at this split.
static int64_t tt_interfaces_doubles(const tt_cores* c, int split) {
  const int d = c->d;
  int64_t tot = 0, Rp = c->n[0];
  tot += Rp * c->r[1];
  for (int k = 1; k < split; ++k) {
    Rp *= c->n[k];
    tot += Rp * c->r[k + 1];
  }
  int64_t Ck = c->n[d - 1];
  tot += Ck * c->r[d - 1];
  for (int k = d - 2; k >= split; --k) {
    Ck *= c->n[k];
    tot += Ck * c->r[k];
  }
  return tot;
}

// The interface levels built into ws (tt_interfaces_doubles of them): *Lout
// (R_split x r_split) points into ws or at a core; the right interface goes to
// Rp with RK >= r_split rows per column, zero past r_split.
static hipError_t tt_interfaces_in(const tt_cores* c, int split, double* ws, int RK, double* Rp, double** Lout,
                                   hipStream_t s) {
  const int d = c->d;
  double* cur = ws;
  int64_t rows = c->n[0], Ck = c->n[d - 1];
  double* L = c->core[0];       // L_1 = G_1 (read only)
  double* R = c->core[d - 1];   // Rt_d = G_d (read only)
  const int nl = split - 1, nr = d - 1 - split;   // levels of each chain
  for (int j = 0; j < std::max(nl, nr); ++j) {
    IfaceLevel A = {};
    if (j < nl) {
      const int k = j + 1;
      A.Lp = L;
      A.Gl = c->core[k];
      A.L = cur;
      A.Rp = rows;
      A.rpl = c->r[k];
      A.nl = (int)c->n[k];
      A.rkl = c->r[k + 1];
      rows *= c->n[k];
      cur += rows * c->r[k + 1];
      A.gl = grid_for(rows, 256);
      L = A.L;
    }
    if (j < nr) {
      const int k = d - 2 - j;
      const bool last = j == nr - 1;
      A.Gr = c->core[k];
      A.Rn = R;
      A.Ck = Ck;
      A.rpr = c->r[k];
      A.nr = (int)c->n[k];
      A.rkr = c->r[k + 1];
      A.ldr = last ? RK : c->r[k];
      Ck *= c->n[k];
      A.Rt = last ? Rp : cur;
      if (!last) cur += Ck * c->r[k];
      A.gr = grid_for(Ck * A.ldr, 256);
      R = A.Rt;
    }
    launch_ifaces(A, s);
  }
  if (nr == 0)
    hipLaunchKernelGGL(k_pad_rt, dim3(grid_for(RK * Ck, 256)), dim3(256), 0, s, R, c->r[d - 1], RK, Ck, Rp);
  *Lout = L;
  return hipGetLastError();
}

// ---- tt_error: one streaming pass over X ----
// Block = 4 waves; a wave owns 128 consecutive rows (2 per lane) of X_m and
// walks the block's column range.  PAIR (R even): a lane's two rows are one
// aligned 2-element load.  The loop body has no branches: lanes past the last
// row read a valid row and drop it (their L rows are zero).  Rt comes padded
// to RK rows with zeros, so a column's RK entries are one contiguous run (wide
// scalar loads).  Eight columns per step keep
// eight loads in flight; every lane still adds its columns in increasing order.
// FN: X is the Hilbert tensor, X(row, col) = fn_rec[fn_row[row] + fn_col[col]],
// evaluated in place of the loads.
struct FnTabs {
  const double* rec;
  const int32_t* row;
  const int32_t* col;
};

template <typename T, int RK, bool PAIR, bool FN>
__global__ __launch_bounds__(256) void k_tt_error(const T* __restrict__ x, int64_t R, int64_t C, int r,
                                                  const double* __restrict__ L, const double* __restrict__ Rt,
                                                  int gi_count, int gj_count, double* __restrict__ part,
                                                  const FnTabs fn) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = blockIdx.x % gi_count, gj = blockIdx.x / gi_count;
  const int64_t row = (int64_t)gi * 512 + w * 128 + 2 * lane;
  const int64_t cb = gj * C / gj_count, ce = (gj + 1) * C / gj_count;
  const bool ok0 = row < R, ok1 = row + 1 < R;
  double l0[RK], l1[RK];
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    l0[k] = (ok0 && k < r) ? L[(int64_t)k * R + row] : 0.0;
    l1[k] = (ok1 && k < r) ? L[(int64_t)k * R + row + 1] : 0.0;
  }
  // rows read by this lane (clamped into the matrix; dropped via w0, w1)
  const int64_t r0c = ok0 ? row : 0, r1c = ok1 ? row + 1 : 0;
  const double w0 = ok0 ? 1.0 : 0.0, w1 = ok1 ? 1.0 : 0.0;
  int fr0 = 0, fr1 = 0;
  if constexpr (FN) {
    fr0 = fn.row[r0c];
    fr1 = fn.row[r1c];
  }
  auto load2 = [&](int64_t col, double& x0, double& x1) {
    if constexpr (FN) {
      const int fc = fn.col[col];
      x0 = fn.rec[fr0 + fc];
      x1 = fn.rec[fr1 + fc];
    } else if constexpr (PAIR) {
      const T* p = x + col * R + r0c;
      if constexpr (sizeof(T) == 8) {
        const double2 v = *(const double2*)p;
        x0 = v.x;
        x1 = v.y;
      } else {
        const float2 v = *(const float2*)p;
        x0 = v.x;
        x1 = v.y;
      }
    } else {
      x0 = (double)x[col * R + r0c];
      x1 = (double)x[col * R + r1c];
    }
    x0 *= w0;
    x1 *= w1;
  };
  double e2 = 0.0, x2 = 0.0;
  auto accum = [&](int64_t col, double x0, double x1) {
    const double* rc = Rt + (int64_t)RK * col;
    double t0 = 0.0, t1 = 0.0;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      const double rv = rc[k];
      t0 += l0[k] * rv;
      t1 += l1[k] * rv;
    }
    const double d0 = x0 - t0, d1 = x1 - t1;
    e2 += d0 * d0 + d1 * d1;
    x2 += x0 * x0 + x1 * x1;
  };
  constexpr int U = 8;
  int64_t col = cb;
  for (; col + U <= ce; col += U) {
    double xa[U], xb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) load2(col + u, xa[u], xb[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) accum(col + u, xa[u], xb[u]);
  }
  for (; col < ce; ++col) {
    double a0, a1;
    load2(col, a0, a1);
    accum(col, a0, a1);
  }
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
    part[2 * blockIdx.x] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    part[2 * blockIdx.x + 1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
  }
}

// Fixed-order sum of nb (e2, x2) pairs: strided per thread, then a tree.
// out[0..1] = (e2, x2); with rel, out[0..2] = (relative error, e2, x2), the
// relative error by the host rule (sqrt(e2 / x2); for x2 = 0: 0 if e2 = 0,
// else +inf).
__global__ __launch_bounds__(256) void k_sum_parts(const double* __restrict__ part, int nb, double* __restrict__ out,
                                                   bool rel) {
  __shared__ double sa[256], sb[256];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sa[threadIdx.x] += sa[threadIdx.x + o];
      sb[threadIdx.x] += sb[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int o = rel ? 1 : 0;
    out[o] = sa[0];
    out[o + 1] = sb[0];
    if (rel) out[0] = sb[0] > 0.0 ? sqrt(sa[0] / sb[0]) : (sa[0] > 0.0 ? INFINITY : 0.0);
  }
}

static int rk_slot(int r) { return r <= 4 ? 4 : r <= 8 ? 8 : r <= 12 ? 12 : r <= 16 ? 16 : r <= 24 ? 24 : 32; }

template <typename T, bool PAIR, bool FN>
static hipError_t launch_err_p(const T* x, int64_t R, int64_t C, int r, const double* L, const double* Rt, int gi,
                               int gj, double* part, const FnTabs& fn, hipStream_t s) {
  dim3 g((unsigned)(gi * gj)), b(256);
  if (r <= 4) hipLaunchKernelGGL((k_tt_error<T, 4, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  else if (r <= 8) hipLaunchKernelGGL((k_tt_error<T, 8, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  else if (r <= 12)
    hipLaunchKernelGGL((k_tt_error<T, 12, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  else if (r <= 16)
    hipLaunchKernelGGL((k_tt_error<T, 16, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  else if (r <= 24)
    hipLaunchKernelGGL((k_tt_error<T, 24, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  else hipLaunchKernelGGL((k_tt_error<T, 32, PAIR, FN>), g, b, 0, s, x, R, C, r, L, Rt, gi, gj, part, fn);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_err(const T* x, int64_t R, int64_t C, int r, const double* L, const double* Rt, int gi,
                             int gj, double* part, hipStream_t s) {
  // aligned pair loads need an even column length (and an aligned base)
  const bool pair = (R % 2) == 0 && ((uintptr_t)x % (2 * sizeof(T))) == 0;
  const FnTabs none{nullptr, nullptr, nullptr};
  return pair ? launch_err_p<T, true, false>(x, R, C, r, L, Rt, gi, gj, part, none, s)
              : launch_err_p<T, false, false>(x, R, C, r, L, Rt, gi, gj, part, none, s);
}

// Geometry and scratch of one error pass over X_m at the middle split.
struct ErrPlan {
  int split, r, RK, gi, gj;
  int64_t R, C;
  int64_t n_iface, n_part, n_rp;   // doubles of the interfaces, the partials (+ the 3 results), padded Rt
};

static ErrPlan err_plan(const tt_cores* c) {
  ErrPlan p;
  const int d = c->d;
  p.split = (d + 1) / 2;
  p.R = p.C = 1;
  for (int k = 0; k < p.split; ++k) p.R *= c->n[k];
  for (int k = p.split; k < d; ++k) p.C *= c->n[k];
  p.r = c->r[p.split];
  p.RK = rk_slot(p.r);
  p.gi = (int)((p.R + 511) / 512);
  p.gj = (int)std::max<int64_t>(1, std::min<int64_t>(p.C, (4096 + p.gi - 1) / p.gi));
  p.n_iface = tt_interfaces_doubles(c, p.split);
  p.n_part = 2 * (int64_t)p.gi * p.gj + 3;
  p.n_rp = (int64_t)p.RK * p.C;
  return p;
}

// The pass itself into caller-provided scratch: interfaces, padded Rt, the
// workgroup partials and their fixed-order sum at out: (e2, x2), or with rel
// (relative error, e2, x2).
// Every scratch entry is written before it is read: nothing needs clearing.
static hipError_t err_launch(const tt_cores* c, const ErrPlan& p, const void* x, int dtype, const FnTabs& fn,
                             double* iface, double* part, double* Rp, double* out, bool rel, hipStream_t s) {
  double* L = nullptr;
  hipError_t e = tt_interfaces_in(c, p.split, iface, p.RK, Rp, &L, s);
  if (e != hipSuccess) return e;
  if (fn.rec) e = launch_err_p<double, false, true>(nullptr, p.R, p.C, p.r, L, Rp, p.gi, p.gj, part, fn, s);
  else if (dtype == PSTT2_F64) e = launch_err((const double*)x, p.R, p.C, p.r, L, Rp, p.gi, p.gj, part, s);
  else e = launch_err((const float*)x, p.R, p.C, p.r, L, Rp, p.gi, p.gj, part, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, s, part, p.gi * p.gj, out, rel);
  return hipGetLastError();
}

// x == nullptr: the Hilbert tensor (fn != 0), evaluated from its index tables
hipError_t tt_error_run(const tt_cores* c, const void* x, int dtype, double* e2x2, hipStream_t s, int fn) {
  const ErrPlan p = err_plan(c);
  double *iface = nullptr, *part = nullptr, *Rp = nullptr, *rec = nullptr;
  int32_t *row_t = nullptr, *col_t = nullptr;
  hipError_t e = ws_alloc((void**)&iface, sizeof(double) * std::max<int64_t>(p.n_iface, 1), s);
  if (e == hipSuccess) e = ws_alloc((void**)&part, sizeof(double) * p.n_part, s);
  if (e == hipSuccess) e = ws_alloc((void**)&Rp, sizeof(double) * p.n_rp, s);
  if (fn) {
    if (e == hipSuccess) e = ws_alloc((void**)&rec, sizeof(double) * hilbert_rec_len(c->n, c->d), s);
    if (e == hipSuccess) e = ws_alloc((void**)&row_t, sizeof(int32_t) * p.R, s);
    if (e == hipSuccess) e = ws_alloc((void**)&col_t, sizeof(int32_t) * p.C, s);
    if (e == hipSuccess) e = hilbert_tables(c->n, c->d, p.split, p.R, p.C, rec, row_t, col_t, s);
  }
  double* out = part ? part + 2 * (int64_t)p.gi * p.gj : nullptr;
  if (e == hipSuccess) e = err_launch(c, p, x, dtype, FnTabs{rec, row_t, col_t}, iface, part, Rp, out, false, s);
  if (e == hipSuccess) e = hipMemcpyAsync(e2x2, out, 2 * sizeof(double), hipMemcpyDeviceToHost, s);
  if (part) ws_free(part, s);
  if (Rp) ws_free(Rp, s);
  if (rec) ws_free(rec, s);
  if (row_t) ws_free(row_t, s);
  if (col_t) ws_free(col_t, s);
  if (iface) ws_free(iface, s);
  hipError_t e2 = hipStreamSynchronize(s);
  return e != hipSuccess ? e : e2;
}

// ---- the same pass with no allocation (tt_error_noalloc) ----
// The scratch is one file-scope device array.  Host code never uses its name as
// an address: the device address comes from hipGetSymbolAddress, once per
// device (each device holds its own copy), and only that pointer reaches the
// kernels.  Calls that overlap on one device share the array and race.
static __device__ __align__(256) unsigned char scratch[PSTT2_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

hipError_t scratch_base(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

int64_t align_doubles(int64_t n) { return (n + 31) / 32 * 32; }   // 256-byte steps
}  // namespace

// Bytes of static scratch an error pass of these cores needs.
int64_t tt_error_scratch_bytes(const tt_cores* c) {
  const ErrPlan p = err_plan(c);
  return 8 * (align_doubles(std::max<int64_t>(p.n_iface, 1)) + align_doubles(p.n_part) + align_doubles(p.n_rp));
}

hipError_t tt_error_noalloc_run(const tt_cores* c, const void* x, int dtype, double* err_dev, hipStream_t s) {
  const ErrPlan p = err_plan(c);
  void* base = nullptr;
  hipError_t e = scratch_base(&base);
  if (e != hipSuccess) return e;
  double* iface = (double*)base;
  double* part = iface + align_doubles(std::max<int64_t>(p.n_iface, 1));
  double* Rp = part + align_doubles(p.n_part);
  // the three results go straight to the caller's buffer
  return err_launch(c, p, x, dtype, FnTabs{nullptr, nullptr, nullptr}, iface, part, Rp, err_dev, true, s);
}

// The Gaussian-bump tensor: its tiles are evaluated on the matrix cores and
// compared with the train's in place (gauss_error), the workgroup partials
// summed in one fixed-order pass.
hipError_t tt_error_run_gauss(const tt_cores* c, const double* centers_host, int nterms, double gamma,
                              double* e2x2, hipStream_t s) {
  const ErrPlan p = err_plan(c);
  double *tabs = nullptr, *iface = nullptr, *part = nullptr, *Rp = nullptr, *L = nullptr;
  GaussTabs g = {};
  int64_t np = 0;
  hipError_t e = ws_alloc((void**)&tabs, sizeof(double) * gauss_table_doubles(c->n, c->d, p.split, nterms), s);
  if (e == hipSuccess) e = gauss_tables(c->n, c->d, p.split, centers_host, nterms, gamma, tabs, &g, s);
  if (e == hipSuccess) {
    np = gauss_error_parts(g);
    e = ws_alloc((void**)&iface, sizeof(double) * std::max<int64_t>(p.n_iface, 1), s);
  }
  if (e == hipSuccess) e = ws_alloc((void**)&part, sizeof(double) * 2 * (np + 1), s);
  if (e == hipSuccess) e = ws_alloc((void**)&Rp, sizeof(double) * p.n_rp, s);
  if (e == hipSuccess) e = tt_interfaces_in(c, p.split, iface, p.RK, Rp, &L, s);
  if (e == hipSuccess) e = gauss_error(g, L, Rp, p.r, p.RK, part, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, s, part, (int)np, part + 2 * np, false);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(e2x2, part + 2 * np, 2 * sizeof(double), hipMemcpyDeviceToHost, s);
  ws_free(part, s);
  ws_free(Rp, s);
  ws_free(iface, s);
  ws_free(tabs, s);
  hipError_t e2 = hipStreamSynchronize(s);
  return e != hipSuccess ? e : e2;
}

// Entries [first, first + count) of X~ = L Rt.  A lane keeps V rows of L in
// registers and walks its workgroup's share of the columns; a column's Rt
// entries are one wave-uniform run (Rt padded to RK rows).  VEC: the V rows are
// consecutive and leave as one 16-byte (V = 2 floats: 8-byte) store; needs R,
// first and count to be multiples of V and an aligned output.  Otherwise they
// are 64 apart, one scalar store each, still contiguous over the wave.
// Every entry sums its ranks in increasing order.
// HBM bound (the output): 4.3 GB of FP32 at R = 64^3, rank 4 slots: one thread
// per entry, with a 64-bit division and 2 r cached loads each, took 2.25 ms;
// this takes 0.82 ms (5.2 TB/s).
template <typename T, int RK, int V, bool VEC>
__global__ __launch_bounds__(256) void k_reconstruct(T* __restrict__ out, int64_t first, int64_t count, int64_t R,
                                                     int64_t c0, int64_t ncol, int r, const double* __restrict__ L,
                                                     const double* __restrict__ Rp, int64_t gi0, int gi_count,
                                                     int gj_count) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = blockIdx.x % gi_count, gj = blockIdx.x / gi_count;
  const int64_t row0 = ((gi0 + gi) * 4 + w) * (64 * V) + (VEC ? V * lane : lane);
  constexpr int ST = VEC ? 1 : 64;
  double l[V][RK];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int64_t row = row0 + ST * v;
#pragma unroll
    for (int k = 0; k < RK; ++k) l[v][k] = (row < R && k < r) ? L[(int64_t)k * R + row] : 0.0;
  }
  const int64_t cb = c0 + gj * ncol / gj_count, ce = c0 + (gj + 1) * ncol / gj_count;
#pragma unroll 4
  for (int64_t col = cb; col < ce; ++col) {
    const double* rc = Rp + (int64_t)RK * col;
    double t[V];
#pragma unroll
    for (int v = 0; v < V; ++v) t[v] = 0.0;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      const double rv = rc[k];
#pragma unroll
      for (int v = 0; v < V; ++v) t[v] += l[v][k] * rv;
    }
    const int64_t f = col * R + row0 - first;
    if constexpr (VEC) {
      if (row0 < R && f >= 0 && f < count) {
        typedef T vec __attribute__((ext_vector_type(V)));
        vec o;
#pragma unroll
        for (int v = 0; v < V; ++v) o[v] = (T)t[v];
        *(vec*)(out + f) = o;
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (row0 + ST * v < R && f + ST * v >= 0 && f + ST * v < count) out[f + ST * v] = (T)t[v];
    }
  }
}

template <typename T, int RK>
static void launch_rec(T* out, int64_t first, int64_t count, int64_t R, int r, const double* L, const double* Rp,
                       hipStream_t s) {
  // rows per lane: 16-byte stores, fewer where the rank's register slots leave no room for four
  constexpr int V = sizeof(T) == 4 && RK <= 16 ? 4 : 2;
  const bool vec = R % V == 0 && first % V == 0 && count % V == 0 && (uintptr_t)out % (V * sizeof(T)) == 0;
  const int64_t c0 = first / R, ncol = (first + count + R - 1) / R - c0;
  const int64_t blocks = (R + 256 * V - 1) / (256 * V);
  constexpr int64_t kMaxBlocks = 1 << 22;   // a launch has less than 2^32 threads
  for (int64_t b0 = 0; b0 < blocks; b0 += kMaxBlocks) {
    const int gi = (int)std::min(blocks - b0, kMaxBlocks);
    // About 4096 workgroups, but shares of eight columns (a lane's V RK loads of L serve its
    // share) while 512 remain: 40^4 FP32 at rank 16 took 97 us with shares of one column,
    // 48 of three.
    const auto shares = [&](int64_t wgs) { return std::min<int64_t>(ncol, (wgs + gi - 1) / gi); };
    const int gj = (int)std::max(shares(512), std::min(shares(4096), ncol / 8));
    const dim3 g((unsigned)gi * gj), b(256);
    if (vec)
      hipLaunchKernelGGL((k_reconstruct<T, RK, V, true>), g, b, 0, s, out, first, count, R, c0, ncol, r, L, Rp, b0, gi,
                         gj);
    else
      hipLaunchKernelGGL((k_reconstruct<T, RK, V, false>), g, b, 0, s, out, first, count, R, c0, ncol, r, L, Rp, b0,
                         gi, gj);
  }
}

template <typename T>
static void launch_rec_r(int RK, T* out, int64_t first, int64_t count, int64_t R, int r, const double* L,
                         const double* Rp, hipStream_t s) {
  switch (RK) {
    case 4: launch_rec<T, 4>(out, first, count, R, r, L, Rp, s); break;
    case 8: launch_rec<T, 8>(out, first, count, R, r, L, Rp, s); break;
    case 12: launch_rec<T, 12>(out, first, count, R, r, L, Rp, s); break;
    case 16: launch_rec<T, 16>(out, first, count, R, r, L, Rp, s); break;
    case 24: launch_rec<T, 24>(out, first, count, R, r, L, Rp, s); break;
    default: launch_rec<T, 32>(out, first, count, R, r, L, Rp, s); break;
  }
}

int64_t tt_reconstruct_doubles(const tt_cores* c) {
  const ErrPlan p = err_plan(c);
  return p.n_iface + p.n_rp;
}

hipError_t tt_reconstruct_run(const tt_cores* c, void* out, int dtype, int64_t first, int64_t count, hipStream_t s) {
  const int d = c->d;
  const int split = (d + 1) / 2;
  int64_t R = 1, C = 1;
  for (int k = 0; k < split; ++k) R *= c->n[k];
  for (int k = split; k < d; ++k) C *= c->n[k];
  const int r = c->r[split], RK = rk_slot(r);
  double *L = nullptr, *ifb = nullptr, *Rp = nullptr;
  hipError_t e = ws_alloc((void**)&ifb, sizeof(double) * tt_interfaces_doubles(c, split), s);
  if (e == hipSuccess) e = ws_alloc((void**)&Rp, sizeof(double) * RK * C, s);
  if (e == hipSuccess) e = tt_interfaces_in(c, split, ifb, RK, Rp, &L, s);
  if (e == hipSuccess && count > 0) {
    if (dtype == PSTT2_F64) launch_rec_r(RK, (double*)out, first, count, R, r, L, Rp, s);
    else launch_rec_r(RK, (float*)out, first, count, R, r, L, Rp, s);
    e = hipGetLastError();
  }
  ws_free(Rp, s);
  ws_free(ifb, s);
  hipError_t e2 = hipStreamSynchronize(s);
  return e != hipSuccess ? e : e2;
}

}  // namespace pstt2
