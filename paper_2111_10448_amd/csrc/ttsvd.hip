// Parallel-TTSVD (Section 3.1, Algorithm Parallel-TTSVD, Theorem perf_alg1):
// a truncated SVD of every unfolding X_k, then the cores from neighbouring
// left singular bases by equation "core".
//
// The SVD of an unfolding is taken by one-sided (Hestenes) Jacobi on its short
// side, directly on the data (no Gram matrix, so the singular values keep
// their relative accuracy): with s = min(R_k, C_k) and L = max(R_k, C_k), the
// work matrix W (L x s) is X_k^T when R_k <= C_k and X_k otherwise.  Pairs of
// columns are rotated until every pair is orthogonal to working precision; J
// (s x s) accumulates the rotations, so W J = W' has orthogonal columns whose
// norms are the singular values.  For W = X_k^T, J holds the left singular
// vectors of X_k; for W = X_k, they are the normalised columns of W'.
//
// Columns go in blocks of eight; block pairs follow the round-robin (circle)
// schedule, so nb - 1 rounds of nb / 2 disjoint pairs (nb the number of blocks
// rounded up to even, columns past s zero and never stored) meet every pair
// once per sweep.  A workgroup takes a block pair: the 16 x 16 Gram matrix of
// its columns from the data (FP64 matrix cores), one sweep of two-sided Jacobi
// on it, and the accumulated 16 x 16 rotation applied to the 16 columns of W
// and J.  Convergence is judged on the Gram entries formed from the data, the
// same test as for single pairs.  Sums run in a fixed order, so results are
// bitwise repeatable.
//
// One pair of columns per workgroup and launch cost 7.3 us a round, nearly all
// of it launch and reduction latency: 4847 rounds, 35 ms, on (20, 17, 19, 21).
// A round of block pairs costs 17 us and stands for about eight of those (383
// rounds, 6.6 ms); the whole call went from 37.9 to 8.1 ms.  It is bound by that
// chain: Gram loads, fifteen dependent rounds of angles, the application.
//
// Where the rank rule keeps fewer than kSvdLead columns and a gap follows them, power
// steps on those columns replace the sweeps (see "leading columns" below): 8.1 -> 1.4 ms
// for the same call, a third of it kernels of some 5 us and their launches, the rest
// the reflectors' chain, the leading block's rotations and two readbacks a split.
#include <algorithm>
#include <cmath>

#include "internal.h"
#include "philox.h"

namespace pstt2 {

namespace {
constexpr int kBS = 256;

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kBC = 8;            // columns per block
constexpr int kPC = 2 * kBC;      // columns of a block pair
constexpr int kJT = 1024;         // threads of the block kernels
constexpr int kChunkRows = 2048;  // rows per workgroup at least

// circle method: position 0 fixed, positions 1..s-1 rotate by one per round
__device__ __forceinline__ int rr_elem(int j, int k, int s) { return j == 0 ? 0 : 1 + (j - 1 + k) % (s - 1); }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Pair (w_p, w_q) counts as orthogonal; tau: columns whose squared norms are
// both at most tau need not be (see svd_sweep).  Nor need a column that is cut in any
// case (squared norm at most small) be against one it cannot turn by a rounding: exact
// zeros leave columns of 1e-150 and less whose products underflow.
__device__ __forceinline__ bool needs_rotation(double a, double b, double g, double tol, double tau, double small) {
  const double lo = a < b ? a : b, hi = a < b ? b : a;
  return g != 0.0 && fabs(g) > tol * sqrt(a * b) && hi > tau && !(lo <= small && lo <= 0x1p-104 * hi);
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  return s;
}
}  // namespace

// Partial maxima of |x|, one per workgroup.
constexpr int kMaxParts = 256;
__global__ __launch_bounds__(256) void k_svd_absmax(const double* __restrict__ x, int64_t n, double* __restrict__ part) {
  __shared__ double red[4];
  double m = 0.0;
  int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x;
  constexpr int64_t ST = kMaxParts * 256;
  for (; t + 7 * ST < n; t += 8 * ST) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[t + u * ST];
#pragma unroll
    for (int u = 0; u < 8; ++u) m = fmax(m, fabs(v[u]));
  }
  for (; t < n; t += ST) m = fmax(m, fabs(x[t]));
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// e with 2^e <= max |x| < 2^{e+1} (0 for no, no finite or only zero entries), in every
// thread of the workgroup of 256.  W holds X / 2^e, exactly: Gram entries square the
// entries and the reflectors of W^T W_1 take their fourth power, so rms entries past
// 1e75 overflowed and below 1e-78 left denormal squares, whose reflectors are not
// orthogonal.  The rank rule and the bases do not see the scale; the last core gets it back.
__device__ __forceinline__ int svd_exponent(const double* __restrict__ part, double* red) {
  double m = part[threadIdx.x];
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  return m > 0.0 && isfinite(m) ? ilogb(m) : 0;
}

// The rotations' start with the columns at place: J(r, place[r]) = 1, those past s at
// their own index (place null: the identity).
__device__ __forceinline__ void svd_eye(double* __restrict__ J, int sp, int s, const int* __restrict__ place) {
  const int64_t tot = (int64_t)sp * sp, stride = (int64_t)gridDim.x * gridDim.y * 256;
  for (int64_t t = (blockIdx.x + (int64_t)gridDim.x * blockIdx.y) * 256 + threadIdx.x; t < tot; t += stride) {
    const int r = (int)(t % sp), c = (int)(t / sp);
    J[t] = (place && r < s ? place[r] : r) == c ? 1.0 : 0.0;
  }
}

// W (C x sp, column-major): W(c, place[r]) = X_k(r, c) / 2^e for r < R, zero columns past R
// (place null: the identity).
// 32 x 32 tiles through LDS so both sides are read and written along rows.
__global__ void k_svd_transpose(const double* __restrict__ x, int64_t R, int64_t C, int sp,
                                const double* __restrict__ xmax, const int* __restrict__ place,
                                double* __restrict__ W, double* __restrict__ J) {
  __shared__ double t[32][33], red[4];
  if (J) svd_eye(J, sp, (int)R, place);
  const int e = svd_exponent(xmax, red);
  const int64_t c0 = (int64_t)blockIdx.x * 32, r0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  for (int j = ty; j < 32; j += 8) {
    const int64_t r = r0 + tx, c = c0 + j;
    t[j][tx] = (r < R && c < C) ? ldexp(x[r + R * c], -e) : 0.0;
  }
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    const int64_t c = c0 + tx, r = r0 + j;
    if (c < C && r < sp) W[c + C * (place && r < R ? place[r] : r)] = t[tx][j];
  }
}

// W (R x sp): X_k / 2^e, its column c at place[c] (null: c), and zero columns past C.
__global__ void k_svd_copy(const double* __restrict__ x, int64_t R, int64_t C, int sp, const double* __restrict__ xmax,
                           const int* __restrict__ place, double* __restrict__ W, double* __restrict__ J) {
  __shared__ double red[4];
  if (J) svd_eye(J, sp, (int)C, place);
  const int e = svd_exponent(xmax, red);
  const int64_t tot = R * sp;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const double v = t < R * C ? ldexp(x[t], -e) : 0.0;
    int64_t o = t;
    if (place && t < R * C) {
      const int64_t c = t / R;
      o = t + R * (place[c] - c);
    }
    W[o] = v;
  }
}

// place[j]: column j's position in order of decreasing norm (ties by index); a norm that
// is not a number counts as infinite, so that place is a permutation all the same.
__global__ __launch_bounds__(256) void k_svd_place(const double* __restrict__ sig, int s, int* __restrict__ place) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= s) return;
  const double own = isnan(sig[j]) ? INFINITY : sig[j];
  int p = 0;
#pragma unroll 8
  for (int i = 0; i < s; ++i) {
    const double o = isnan(sig[i]) ? INFINITY : sig[i];
    p += o > own || (o == own && i < j) ? 1 : 0;
  }
  place[j] = p;
}

// Columns of block pair i in round k: column c < 16 of the pair, sp or more if
// there is none.
struct PairCols {
  int b0, b1;
  __device__ __forceinline__ PairCols(int i, int k, int nb) : b0(rr_elem(i, k, nb)), b1(rr_elem(nb - 1 - i, k, nb)) {}
  __device__ __forceinline__ int col(int c) const { return (c < kBC ? b0 : b1) * kBC + (c & (kBC - 1)); }
};

// Gram matrix of the pair's columns over rows [r0, r1), summed over the waves
// into G.  Lane (g4, l16) holds column l16 of rows 8 j + 2 g4 and + 1 of a
// 64-row tile: the same register is both operands of the 16x16x4 product, so
// any assignment of rows to the K index serves.
__device__ __forceinline__ void pair_gram(const double* __restrict__ W, int64_t L, int sp, const PairCols& pc,
                                          int64_t r0, int64_t r1, double (*part)[kPC * kPC], double* G) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int col = pc.col(l16);
  const double* wc = W + (int64_t)(col < sp ? col : 0) * L;
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
  for (int64_t t = r0 + 64 * w; t < r1; t += 64 * (kJT / 64)) {
    double v[16];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int64_t r = t + 8 * j + 2 * g4 + e;
        const bool in = r < r1 && col < sp;
        const double x = wc[in ? r : r0];
        v[2 * j + e] = in ? x : 0.0;
      }
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[j], v[j], acc[j & 1], 0, 0, 0);
  }
  acc[0] += acc[1];
#pragma unroll
  for (int e = 0; e < 4; ++e) part[w][(4 * e + g4) * kPC + l16] = acc[0][e];
  __syncthreads();
  if (threadIdx.x < kPC * kPC) {
    double s = part[0][threadIdx.x];
    for (int ww = 1; ww < kJT / 64; ++ww) s += part[ww][threadIdx.x];
    G[threadIdx.x] = s;
  }
}

// Sweeps of two-sided Jacobi on the Gram matrix G by one wavefront, the
// rotations accumulated into Q.  A round rotates eight disjoint pairs: lane
// (i, j) owns the 2 x 2 block of pair i's rows and pair j's columns, so a round
// is one pass over G.  The chain of a round's dependent steps is what it costs:
// the tangent of an angle comes from the hardware's approximate reciprocal and
// root (1e-7 or better; an inexact angle only leaves a residual that the next
// meeting of the pair removes), the cosine and sine from it in full precision,
// so every rotation is orthogonal to rounding.
__device__ __forceinline__ void pair_sweeps(double (*G)[kPC + 1], double (*Q)[kPC + 1], double tol, double tau,
                                            int sweeps) {
  const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
  wave_sync();
  for (int sw = 0; sw < sweeps; ++sw) {
    bool any = false;
    for (int rnd = 0; rnd < kPC - 1; ++rnd) {
      const int p = rr_elem(j, rnd, kPC), q = rr_elem(kPC - 1 - j, rnd, kPC);
      const int pi = rr_elem(i, rnd, kPC), qi = rr_elem(kPC - 1 - i, rnd, kPC);
      const double a = G[p][p], b = G[q][q], g = G[p][q];
      double g00 = G[pi][p], g01 = G[pi][q], g10 = G[qi][p], g11 = G[qi][q];
      double u0 = Q[i][p], v0 = Q[i][q], u1 = Q[i + kBC][p], v1 = Q[i + kBC][q];
      double c = 1.0, s = 0.0;
      // the test of needs_rotation with an approximate root: slightly tighter, so
      // that no pair counted as not orthogonal is passed over here
      const double ab = a * b;
      const double lim = ab > 1e-290 ? ab * __builtin_amdgcn_rsq(ab) : sqrt(ab);
      const bool rot = g != 0.0 && fabs(g) > 0.99 * tol * lim && (a > tau || b > tau);
      if (rot) {
        // tan of the angle that zeroes the off-diagonal entry of [[a, g], [g, b]]
        const double z = 0.5 * (b - a) * __builtin_amdgcn_rcp(g);
        const double az = fabs(z), h = 1.0 + z * z;
        const double t = az < 1e100 ? __builtin_amdgcn_rcp(az + h * __builtin_amdgcn_rsq(h)) : 0.0;
        const double tn = z >= 0.0 ? t : -t;
        const double x = 1.0 + tn * tn;   // in [1, 2]: two Newton steps to full precision
        c = __builtin_amdgcn_rsq(x);
        c += 0.5 * c * fma(-x * c, c, 1.0);
        c += 0.5 * c * fma(-x * c, c, 1.0);
        s = c * tn;
      }
      if (!__any(rot)) continue;
      any = true;
      const double ci = __shfl(c, i), si = __shfl(s, i);   // lane i < 8 holds pair i's angle
      // columns p, q of the block, then rows pi, qi
      double t0 = c * g00 - s * g01, t1 = s * g00 + c * g01;
      g00 = t0;
      g01 = t1;
      t0 = c * g10 - s * g11;
      t1 = s * g10 + c * g11;
      g10 = t0;
      g11 = t1;
      wave_sync();   // every lane has read its entries
      G[pi][p] = ci * g00 - si * g10;
      G[pi][q] = ci * g01 - si * g11;
      G[qi][p] = si * g00 + ci * g10;
      G[qi][q] = si * g01 + ci * g11;
      Q[i][p] = c * u0 - s * v0;
      Q[i][q] = s * u0 + c * v0;
      Q[i + kBC][p] = c * u1 - s * v1;
      Q[i + kBC][q] = s * u1 + c * v1;
      wave_sync();
    }
    if (!any) break;
  }
}

__global__ __launch_bounds__(kJT) void k_jacobi_gram(const double* __restrict__ W, int64_t L, int sp, int nb, int k,
                                                     int64_t chunk, int nch, double* __restrict__ gpart) {
  __shared__ double part[kJT / 64][kPC * kPC];
  const int i = blockIdx.x % (nb / 2), ch = blockIdx.x / (nb / 2);
  const PairCols pc(i, k, nb);
  const int64_t r0 = ch * chunk, r1 = r0 + chunk < L ? r0 + chunk : L;
  pair_gram(W, L, sp, pc, r0, r1, part, gpart + ((int64_t)i * nch + ch) * kPC * kPC);
}

// One block pair of a round: its Gram matrix (formed here when one workgroup
// holds all L rows, else the sum of k_jacobi_gram's partials, the same in every
// workgroup of the pair), the rotation, and its application to this workgroup's
// rows of W and, in the pair's first workgroup, to J.
__global__ __launch_bounds__(kJT) void k_jacobi_blocks(double* __restrict__ W, int64_t L, double* __restrict__ J,
                                                       int jr, int sp, int nb, int k, double tol, double tau,
                                                       double small, int sweeps,
                                                       int64_t chunk, int nch, const double* __restrict__ gpart,
                                                       int* __restrict__ rotations) {
  __shared__ double part[kJT / 64][kPC * kPC];
  __shared__ double G0[kPC * kPC];
  __shared__ double G[kPC][kPC + 1], Q[kPC][kPC + 1];
  __shared__ int todo;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int i = blockIdx.x % (nb / 2), ch = blockIdx.x / (nb / 2);
  const PairCols pc(i, k, nb);
  const int64_t r0 = ch * chunk, r1 = r0 + chunk < L ? r0 + chunk : L;
  if (nch == 1) {
    pair_gram(W, L, sp, pc, r0, r1, part, G0);
  } else if (t < kPC * kPC) {
    double s = 0.0;
    for (int c = 0; c < nch; ++c) s += gpart[((int64_t)i * nch + c) * kPC * kPC + t];
    G0[t] = s;
  }
  __syncthreads();
  if (w == 0) {
    int bad = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int e = lane + 64 * h, r = e / kPC, c = e % kPC;
      G[r][c] = G0[e];
      Q[r][c] = r == c ? 1.0 : 0.0;
      if (r < c && needs_rotation(G0[r * kPC + r], G0[c * kPC + c], G0[e], tol, tau, small)) ++bad;
    }
    for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o);
    if (lane == 0) {
      todo = bad;
      if (bad && ch == 0) atomicAdd(rotations, bad);
    }
    if (bad) pair_sweeps(G, Q, tol, tau, sweeps);
  }
  __syncthreads();
  if (todo == 0) return;   // uniform across the workgroup
  // W(:, pair) <- W(:, pair) Q in 16-row tiles, each read and written by one wave:
  // D = Q^T W^T, operands Q(4 ks + g4, l16) and W(row l16, column 4 ks + g4), element
  // v of the result at new column 4 v + g4, row l16
  double qa[4];
  int64_t ci[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qa[ks] = Q[4 * ks + g4][l16];
    ci[ks] = pc.col(4 * ks + g4);
  }
  // tiles of this workgroup's rows of W, then (first workgroup) those of J; a wave
  // takes kAU tiles at a time, every load before the first store
  const int64_t ntw = (r1 - r0 + 15) / 16, nt = ntw + (ch == 0 ? (jr + 15) / 16 : 0);
  constexpr int kAU = 3;
  for (int64_t t0 = w; t0 < nt; t0 += kAU * (kJT / 64)) {
    double x[kAU][4];
    double* m[kAU];
    int64_t ld[kAU];
#pragma unroll
    for (int u = 0; u < kAU; ++u) {
      const int64_t tt = t0 + u * (kJT / 64);
      const bool inw = tt < ntw;
      const int64_t r = inw ? r0 + 16 * tt + l16 : 16 * (tt - ntw) + l16;
      ld[u] = inw ? L : jr;
      m[u] = tt < nt && r < (inw ? r1 : (int64_t)jr) ? (inw ? W : J) + r : nullptr;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bool ok = m[u] && ci[ks] < sp;
        const double v = ok ? m[u][ci[ks] * ld[u]] : 0.0;
        x[u][ks] = v;
      }
    }
#pragma unroll
    for (int u = 0; u < kAU; ++u) {
      d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[ks], x[u][ks], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (m[u] && ci[v] < sp) m[u][ci[v] * ld[u]] = acc[v];
    }
  }
}

// ---- leading columns ----
// Where the rank rule cuts a tail that a gap sets off, only the pairs with a kept
// column matter, and sweeps meet them a block at a time.  Turning the columns by an
// orthogonal H whose first sixteen columns span those of W^T W_1 (W_1 the first
// sixteen of W; at first W Omega, Omega random) is a power step for all of them at
// once: W <- W H, J <- J H, H = I - V T V^T from the reflectors of W^T W_1.  It stays
// orthogonal to rounding; with the sixteen made orthogonal among themselves the test of
// the sweeps is met by every pair with a kept column after a few steps.  Three
// launches, 35 us, a step (17 us for the reflectors of 340 rows, 11 for the turn),
// against seventeen microseconds a round of block pairs.
//
// The columns are first put in order of decreasing norm.  H is then graded as they are
// and a small column gets no rounding of a large one; in any other order the first turn
// mixes them (90 x 24, column norms 1 .. 1e-23 increasing: singular values of 1e-9 to
// 1e-11 of the largest off by 1e-9 to 2e-6, in order 1e-15, as by the sweeps alone).

// Omega (s x kSvdLead), uniform in [-1, 1): entries 4 p .. 4 p + 3 from the Philox block of
// counter p (key 0)
__global__ void k_svd_omega(double* __restrict__ Om, int s) {
  static_assert(kSvdLead % 4 == 0, "whole blocks");
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; 4 * p < s * kSvdLead; p += gridDim.x * blockDim.x) {
    const uint32_t ctr[4] = {(uint32_t)p, 0u, 0u, 0u};
    uint32_t x[4];
    philox4x32_10(ctr, 0u, 0u, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) Om[4 * p + i] = (double)(int32_t)x[i] * 0x1p-31;
  }
}

// M <- M H for the rows of W (L x s) and of J (s x s); a workgroup takes 16 rows, its
// waves share the columns.
__global__ __launch_bounds__(kBS) void k_svd_turn(double* __restrict__ W, int64_t L, double* __restrict__ J, int s,
                                                  const double* __restrict__ V, const double* __restrict__ T,
                                                  int64_t tile0) {
  constexpr int P = kSvdLead, NW = kBS / 64;
  static_assert(P == 16, "one tile");
  __shared__ double part[NW][P][17], MT[P][17], Ts[P][P];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int64_t ntw = (L + 15) / 16;
  const int64_t tile = tile0 + blockIdx.x;
  const bool inw = tile < ntw;
  double* M = inw ? W : J;
  const int64_t ld = inw ? L : s, row = 16 * (inw ? tile : tile - ntw) + l16;
  const bool ok = row < ld;
  auto vx = [&](int j, int c) -> double {   // V with its unit diagonal
    const double v = j < s ? V[(int64_t)c * s + j] : 0.0;
    return j > c ? v : (j == c ? 1.0 : 0.0);
  };
  Ts[t & 15][t >> 4] = T[t];   // [row][column]
  // M V: result element v at column 4 v + g4, row l16
  d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int j0 = 4 * w; j0 < s; j0 += 4 * NW) {
    const int j = j0 + g4;
    const double x = ok && j < s ? M[row + ld * j] : 0.0;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(vx(j, l16), x, acc, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[w][4 * e + g4][l16] = acc[e];
  __syncthreads();
  {
    const int r = t & 15, c = t >> 4;   // (M V T)(r, c)
    double sum = 0.0;
    for (int k = 0; k <= c; ++k) {
      double p = 0.0;
      for (int ww = 0; ww < NW; ++ww) p += part[ww][k][r];
      sum += p * Ts[k][c];
    }
    MT[c][r] = sum;
  }
  __syncthreads();
  double mt[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) mt[k] = MT[4 * k + g4][l16];
#pragma unroll 2
  for (int j0 = 16 * w; j0 < s; j0 += 16 * NW) {
    d4 d = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) d = __builtin_amdgcn_mfma_f64_16x16x4f64(vx(j0 + l16, 4 * k + g4), mt[k], d, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = j0 + 4 * e + g4;
      if (ok && j < s) M[row + ld * j] -= d[e];
    }
  }
}

// Pairs of one of the leading columns (products C = W^T W_1, s x kSvdLead) that the
// sweeps would still rotate.
__global__ void k_svd_lead_check(const double* __restrict__ C, int s, const double* __restrict__ sig, int scols,
                                 double tol, double tau, double small, int* __restrict__ counter) {
  int bad = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < scols * kSvdLead; t += gridDim.x * blockDim.x) {
    const int j = t % scols, i = t / scols;
    if (j > i && needs_rotation(sig[i] * sig[i], sig[j] * sig[j], C[(int64_t)i * s + j], tol, tau, small)) ++bad;
  }
  if (bad) atomicAdd(counter, bad);
}

// sig[j] = ||W(:, j)||, of W / 2^e with xmax, one workgroup per column
__global__ __launch_bounds__(kBS) void k_svd_colnorm(const double* __restrict__ W, int64_t L,
                                                     const double* __restrict__ xmax, double* __restrict__ sig) {
  __shared__ double red[kBS / 64];
  const int e = xmax ? svd_exponent(xmax, red) : 0;
  const double* w = W + (int64_t)blockIdx.x * L;
  double a = 0.0;
  int64_t t = threadIdx.x;
  for (; t + 7 * kBS < L; t += 8 * kBS) {   // eight loads in flight, summed in order
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ldexp(w[t + u * kBS], -e);
#pragma unroll
    for (int u = 0; u < 8; ++u) a += v[u] * v[u];
  }
  for (; t < L; t += kBS) {
    const double v = ldexp(w[t], -e);
    a += v * v;
  }
  a = block_sum(a, red);
  if (threadIdx.x == 0) sig[blockIdx.x] = sqrt(a);
}

// dst (rows x r): dst(:, a) = src(:, idx[a]) / (sig ? sig[idx[a]] : 1), src with
// leading dimension ld.  A kept column with a zero singular value (X = 0) has no
// direction of its own: it becomes the unit vector e_a.
__global__ void k_svd_gather(const double* __restrict__ src, int64_t ld, int64_t rows, const int* __restrict__ idx,
                             const double* __restrict__ sig, int r, double* __restrict__ dst) {
  const int64_t tot = rows * r;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(t / rows);
    const int64_t row = t % rows;
    const int j = idx[a];
    if (!sig) dst[t] = src[(int64_t)j * ld + row];
    else dst[t] = sig[j] > 0.0 ? src[(int64_t)j * ld + row] / sig[j] : (row == a ? 1.0 : 0.0);
  }
}

// Last core from W' = X_{d-1}^T U / 2^e: G(a, i) = 2^e W'(i, idx a) (r x n_d, column-major).
__global__ void k_svd_last_core(const double* __restrict__ src, int64_t ld, const int* __restrict__ idx,
                                const double* __restrict__ xmax, int r, int nd, double* __restrict__ G) {
  __shared__ double red[4];
  const int e = svd_exponent(xmax, red);
  const int64_t tot = (int64_t)r * nd;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(t % r);
    const int i = (int)(t / r);
    G[t] = ldexp(src[(int64_t)idx[a] * ld + i], e);
  }
}

// v <- P^T v for n vectors of r entries (entry a of vector i at a es + i vs): U <- U P is
// orthonormal to the square of what U (columns by decreasing singular value, E = U^T U)
// was, which thousands of rounded rotations leave up to 1e-13 from orthonormal.  P is
// triangular, P^T E P = I to first order: lower, a column takes its correction from those
// of smaller singular values, upper (up) from those of larger ones.  A row of the last
// core changes by rows of smaller singular values only, lower where the core is W'^T
// (P^T W'^T), upper where it is Sigma J^T (P^{-1} Sigma J^T): relative accuracy of small
// rows does not rest on how small E's entries happen to be, as with a symmetric P.
__global__ __launch_bounds__(256) void k_svd_polish(const double* __restrict__ E, int r, bool up, int64_t n, int64_t es,
                                                    int64_t vs, double* __restrict__ V) {
  constexpr int MX = PSTT2_MAX_ELL;
  __shared__ double Es[MX][MX + 1];
  for (int t = threadIdx.x; t < r * r; t += 256) {
    const int a = t % r, b = t / r;
    Es[a][b] = a == b ? 1.5 - 0.5 * E[t] : ((b < a) == up ? -E[t] : 0.0);
  }
  __syncthreads();
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    double v[MX];
#pragma unroll
    for (int a = 0; a < MX; ++a) v[a] = a < r ? V[a * es + i * vs] : 0.0;
    for (int a = 0; a < r; ++a) {
      double s = 0.0;
#pragma unroll
      for (int b = 0; b < MX; ++b)
        if (b < r) s += Es[a][b] * v[b];
      V[a * es + i * vs] = s;
    }
  }
}

// Rows a0 .. r - 1 of the last core from J: 2^e P^{-1} Sigma J^T with the upper P of
// k_svd_polish, to first order.
__global__ __launch_bounds__(256) void k_svd_small_rows(const double* __restrict__ J, int sp,
                                                        const double* __restrict__ E, const double* __restrict__ sig,
                                                        const int* __restrict__ idx, const double* __restrict__ xmax,
                                                        int r, int a0, int nd, double* __restrict__ G) {
  __shared__ double red[4];
  const int e = svd_exponent(xmax, red);
  const int64_t tot = (int64_t)(r - a0) * nd;
  for (int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x; t < tot; t += (int64_t)gridDim.x * 256) {
    const int a = a0 + (int)(t / nd);
    const int64_t i = t % nd;
    double s = 0.0;
    for (int b = a; b < r; ++b)
      s += (b == a ? 0.5 + 0.5 * E[a + r * a] : E[a + r * b]) * (sig[idx[b]] * J[(int64_t)idx[b] * sp + i]);
    G[a + (int64_t)r * i] = ldexp(s, e);
  }
}

__global__ void k_zero_int(int* p) { *p = 0; }

static unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }

int svd_max_parts() { return kMaxParts; }

hipError_t svd_absmax(const double* x, int64_t n, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_absmax, dim3(kMaxParts), dim3(256), 0, s, x, n, part);
  return hipGetLastError();
}

hipError_t svd_load(const double* x, int64_t R, int64_t C, int sp, const double* xmax, const int* place, double* W,
                    double* J, hipStream_t s) {
  if (R <= C) {
    const dim3 g((unsigned)((C + 31) / 32), (unsigned)((sp + 31) / 32));
    hipLaunchKernelGGL(k_svd_transpose, g, dim3(256), 0, s, x, R, C, sp, xmax, place, W, J);
  } else {
    hipLaunchKernelGGL(k_svd_copy, dim3(grid_of(R * sp)), dim3(256), 0, s, x, R, C, sp, xmax, place, W, J);
  }
  return hipGetLastError();
}

hipError_t svd_place(const double* sig, int scols, int* place, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_place, dim3((unsigned)((scols + 255) / 256)), dim3(256), 0, s, sig, scols, place);
  return hipGetLastError();
}

static int svd_chunks(int64_t L, int64_t* chunk) {
  const int64_t nch = std::min<int64_t>(64, (L + kChunkRows - 1) / kChunkRows);
  *chunk = ((L + nch - 1) / nch + 63) / 64 * 64;
  return (int)((L + *chunk - 1) / *chunk);
}

static int svd_blocks(int sp) { return std::max(2, ((sp + kBC - 1) / kBC + 1) / 2 * 2); }

int64_t svd_ws_doubles(int64_t L, int sp) {
  int64_t chunk = 0;
  const int nch = svd_chunks(L, &chunk);
  return nch > 1 ? (int64_t)svd_blocks(sp) / 2 * nch * kPC * kPC : 0;
}

hipError_t svd_sweep(double* W, int64_t L, double* J, int jr, int sp, double tol, double tau, double small, double* ws,
                     int* counter, hipStream_t s) {
  int64_t chunk = 0;
  const int nch = svd_chunks(L, &chunk), nb = svd_blocks(sp);
  const int sweeps = nb == 2 ? 8 : 1;   // a single pair of blocks: to convergence on its Gram matrix
  const dim3 g((unsigned)(nb / 2 * nch)), b(kJT);
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, s, counter);
  for (int k = 0; k < nb - 1; ++k) {
    if (nch > 1) hipLaunchKernelGGL(k_jacobi_gram, g, b, 0, s, W, L, sp, nb, k, chunk, nch, ws);
    hipLaunchKernelGGL(k_jacobi_blocks, g, b, 0, s, W, L, J, jr, sp, nb, k, tol, tau, small, sweeps, chunk, nch, ws, counter);
  }
  return hipGetLastError();
}

// lead: products C (sp x P), reflectors V (sp x P), T and R (P x P each), W Omega (L x P)
int64_t svd_lead_doubles(int64_t L, int sp) {
  return (int64_t)kSvdLead * (2 * (int64_t)sp + 2 * kSvdLead + L);
}

hipError_t svd_lead_turn(double* W, int64_t L, double* J, int sp, double* lead, hipStream_t s) {
  double *V = lead + (int64_t)sp * kSvdLead, *T = V + (int64_t)sp * kSvdLead;
  hipError_t e = qr_reflectors(lead, sp, V, T, T + kSvdLead * kSvdLead, s);
  if (e != hipSuccess) return e;
  const int64_t tiles = (L + 15) / 16 + (sp + 15) / 16;
  constexpr int64_t kMaxGrid = 1 << 23;   // workgroups of a launch: 2^32 threads wrap around
  for (int64_t t0 = 0; t0 < tiles; t0 += kMaxGrid)
    hipLaunchKernelGGL(k_svd_turn, dim3((unsigned)std::min(tiles - t0, kMaxGrid)), dim3(kBS), 0, s, W, L, J, sp, V, T, t0);
  return hipGetLastError();
}

// C = W^T W_1
hipError_t svd_lead_products(const double* W, int64_t L, int sp, double* lead, hipStream_t s) {
  return adj_gemm(true, false, sp, kSvdLead, L, 1.0, W, L, W, L, 0.0, lead, sp, s);
}

// First turn, from W^T (W Omega).
hipError_t svd_lead_init(double* W, int64_t L, double* J, int sp, double* lead, hipStream_t s) {
  double* Z = lead + (int64_t)kSvdLead * (2 * (int64_t)sp + 2 * kSvdLead);
  double* Om = lead + (int64_t)sp * kSvdLead;   // where the reflectors go
  hipLaunchKernelGGL(k_svd_omega, dim3(grid_of((int64_t)sp * kSvdLead / 4)), dim3(256), 0, s, Om, sp);
  hipError_t e = adj_gemm(false, false, L, kSvdLead, sp, 1.0, W, L, Om, sp, 0.0, Z, L, s);
  if (e == hipSuccess) e = adj_gemm(true, false, sp, kSvdLead, L, 1.0, W, L, Z, L, 0.0, lead, sp, s);
  if (e == hipSuccess) e = svd_lead_turn(W, L, J, sp, lead, s);
  return e;
}

hipError_t svd_lead_check(const double* sig, int scols, int sp, const double* lead, double tol, double tau, double small,
                          int* counter, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, s, counter);
  hipLaunchKernelGGL(k_svd_lead_check, dim3(grid_of((int64_t)scols * kSvdLead)), dim3(256), 0, s, lead, sp, sig,
                     scols, tol, tau, small, counter);
  return hipGetLastError();
}

hipError_t svd_colnorms(const double* W, int64_t L, int scols, const double* xmax, double* sig, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_colnorm, dim3((unsigned)scols), dim3(kBS), 0, s, W, L, xmax, sig);
  return hipGetLastError();
}

hipError_t svd_gather(const double* src, int64_t ld, int64_t rows, const int* idx, const double* sig, int r,
                      double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_gather, dim3(grid_of(rows * r)), dim3(256), 0, s, src, ld, rows, idx, sig, r, dst);
  return hipGetLastError();
}

hipError_t svd_last_core(const double* src, int64_t ld, const int* idx, const double* xmax, int r, int nd, double* G,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_svd_last_core, dim3(grid_of((int64_t)r * nd)), dim3(256), 0, s, src, ld, idx, xmax, r, nd, G);
  return hipGetLastError();
}

hipError_t svd_polish(const double* E, int r, bool up, int64_t n, int64_t es, int64_t vs, double* V, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_polish, dim3(grid_of(n)), dim3(256), 0, s, E, r, up, n, es, vs, V);
  return hipGetLastError();
}

hipError_t svd_small_rows(const double* J, int sp, const double* E, const double* sig, const int* idx,
                          const double* xmax, int r, int a0, int nd, double* G, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_small_rows, dim3(grid_of((int64_t)(r - a0) * nd)), dim3(256), 0, s, J, sp, E, sig, idx, xmax, r,
                     a0, nd, G);
  return hipGetLastError();
}

}  // namespace pstt2
