// Small dense FP64 products of the recovery and the adjoint, column-major, on
// FP64 matrix cores.  Operand layout of the 16x16x4 instruction: lane (g4, l16)
// holds element (l16, g4) of A (M x K) and element (g4, l16) of B (K x N);
// element v of the result sits at (4 v + g4, l16).
#include <algorithm>

#include "internal.h"

namespace pstt2 {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wsum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ double at(const double* A, int64_t lda, bool t, int64_t i, int64_t k) {
  return t ? A[k + lda * i] : A[i + lda * k];
}

// Workgroups of a launch at most: one of 2^32 threads is refused, one of more wraps
// around.  Larger grids go in several launches, blk0 the first workgroup of each.
constexpr int64_t kMaxGrid = 1 << 23;

// ---- C = alpha op(A) op(B) + beta C, short contractions ----
// A wave forms one 16 x 16 tile of C^T (rows of C on the lanes of a store, so it
// covers 16 consecutive rows), eight inner entries in flight.  SPLIT: the four
// waves of a workgroup share one tile, a quarter of the inner index each, added
// in wave order; else they take four tiles.  Latency bound: the chain per wave
// is K / 4 steps (K / 16 with SPLIT); one thread per entry ran K dependent
// loads (12.9 us a call on average in the adjoint at n = 24^5, K up to 192; now
// 3.8 us).
template <bool SPLIT>
__global__ __launch_bounds__(256) void k_gemm_m(bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
                                                const double* __restrict__ A, int64_t lda, const double* __restrict__ B,
                                                int64_t ldb, double beta, double* __restrict__ C, int64_t ldc,
                                                int64_t blk0) {
  __shared__ double red[SPLIT ? 4 : 1][SPLIT ? 256 : 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int64_t mt = (M + 15) / 16, ntile = mt * ((N + 15) / 16);
  const int64_t tile = SPLIT ? blk0 + blockIdx.x : (blk0 + blockIdx.x) * 4 + w;
  if (!SPLIT && tile >= ntile) return;
  const int64_t i0 = tile % mt * 16, j0 = tile / mt * 16;
  const int64_t i = i0 + l16 < M ? i0 + l16 : M - 1, j = j0 + l16 < N ? j0 + l16 : N - 1;
  int64_t k0 = 0, k1 = K;
  if constexpr (SPLIT) {
    k0 = (w * K / 4 + 3) / 4 * 4;
    k1 = w == 3 ? K : ((w + 1) * K / 4 + 3) / 4 * 4;
  }
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
  for (int64_t k = k0; k < k1; k += 8) {
    double a[2], b[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t kk = k + 4 * u + g4;
      const bool in = kk < k1;
      const int64_t kc = in ? kk : k0;
      a[u] = at(A, lda, ta, i, kc);
      b[u] = at(B, ldb, !tb, j, kc);
      a[u] = in ? a[u] : 0.0;
      b[u] = in ? b[u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[u], a[u], acc[u], 0, 0, 0);
  }
  acc[0] += acc[1];
  auto put = [&](int64_t ii, int64_t jj, double s) {
    if (ii < M && jj < N) {
      double* c = C + ii + ldc * jj;
      *c = alpha * s + (beta == 0.0 ? 0.0 : beta * *c);
    }
  };
  if constexpr (SPLIT) {
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w][(4 * v + g4) * 16 + l16] = acc[0][v];
    __syncthreads();
    const int t = threadIdx.x;
    put(i0 + (t & 15), j0 + (t >> 4), red[0][t] + red[1][t] + red[2][t] + red[3][t]);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) put(i0 + l16, j0 + 4 * v + g4, acc[0][v]);
  }
}

// one wavefront per entry of C (long contractions)
__global__ __launch_bounds__(256) void k_gemm_w(bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
                                                const double* __restrict__ A, int64_t lda, const double* __restrict__ B,
                                                int64_t ldb, double beta, double* __restrict__ C, int64_t ldc) {
  const int lane = threadIdx.x & 63;
  const int64_t tot = M * N;
  for (int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6; t < tot;
       t += ((int64_t)gridDim.x * blockDim.x) >> 6) {
    const int64_t i = t % M, j = t / M;
    double s = 0.0;
    for (int64_t k = lane; k < K; k += 64) s += at(A, lda, ta, i, k) * at(B, ldb, !tb, j, k);
    s = wsum(s);
    if (lane == 0) {
      double* c = C + i + ldc * j;
      *c = alpha * s + (beta == 0.0 ? 0.0 : beta * *c);
    }
  }
}

// ---- tall, narrow products C_i = A_i^T B_i, M, N <= 32 ----
// Both operands have their columns on l16 and rows on g4, straight from memory:
// a wave takes 8 rows per step (lane rows 2 g4, 2 g4 + 1, 16 bytes a column
// where aligned), four steps in flight, no LDS until the waves' tiles are added.
// Workgroup (slice, i), the batch index fastest: the products of one row slice
// run together and read a shared A once from HBM.  One slice: the result is
// written; else one partial per slice, added in slice order by k_tn_sum (fixed
// butterfly: deterministic).  HBM bound when tall: at K = 49k x 38 products
// (M = N = 8) the LDS version took 98 us for 0.12 GB, this 52; the middle core's
// Z at 64 products of K = 4096, N = 32 took 80 us in a kernel of its own, now 22.
struct TnArgs {
  int M, N;
  int64_t K;
  const double* A;
  int64_t lda, ra, sa;   // column stride, row stride, batch stride
  const double* B;
  int64_t ldb, rb, sb;
  double alpha, beta;
  double* C;
  int64_t ldc, sc;
  int nbatch, nb;        // products, slices
  int64_t rows;          // rows per slice (a multiple of 32)
  double* part;
  int64_t blk0;
};

template <int MT, int NT, bool PAIR>
__global__ __launch_bounds__(256) void k_tn(const TnArgs P) {
  __shared__ double red[4][MT * NT * 256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int bi = (int)((P.blk0 + blockIdx.x) % P.nbatch);
  const int64_t g = (P.blk0 + blockIdx.x) / P.nbatch;
  const int64_t s0 = g * P.rows, s1 = s0 + P.rows < P.K ? s0 + P.rows : P.K;
  // columns past the last one read it again; their results are dropped
  const double *pa[MT], *pb[NT];
#pragma unroll
  for (int t = 0; t < MT; ++t) pa[t] = P.A + bi * P.sa + (int64_t)(16 * t + l16 < P.M ? 16 * t + l16 : P.M - 1) * P.lda;
#pragma unroll
  for (int t = 0; t < NT; ++t) pb[t] = P.B + bi * P.sb + (int64_t)(16 * t + l16 < P.N ? 16 * t + l16 : P.N - 1) * P.ldb;
  d4 acc[MT][NT];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  const int64_t per = P.rows / 4;   // rows per wave, a multiple of 8
  const int64_t r0 = s0 + w * per, r1 = r0 + per < s1 ? r0 + per : s1;
#pragma unroll 4
  for (int64_t r = r0; r < r1; r += 8) {
    const int64_t ra = r + 2 * g4;
    const bool in0 = ra < r1, in1 = ra + 1 < r1;
    double a[MT][2], b[NT][2];
    auto load = [&](const double* p, int64_t rs, double* o) {
      if constexpr (PAIR) {   // r1 is even: both rows are in or out
        const double2 x = *(const double2*)(p + (in0 ? ra : r0));
        o[0] = in0 ? x.x : 0.0;
        o[1] = in0 ? x.y : 0.0;
      } else {
        const double x = p[(in0 ? ra : r0) * rs], y = p[(in1 ? ra + 1 : r0) * rs];
        o[0] = in0 ? x : 0.0;
        o[1] = in1 ? y : 0.0;
      }
    };
#pragma unroll
    for (int t = 0; t < MT; ++t) load(pa[t], P.ra, a[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) load(pb[t], P.rb, b[t]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[w][(i * NT + j) * 256 + l16 * 16 + 4 * v + g4] = acc[i][j][v];
  __syncthreads();
  const int nout = P.M * P.N;
  for (int o = threadIdx.x; o < nout; o += 256) {
    const int i = o % P.M, j = o / P.M;
    const int e = ((i >> 4) * NT + (j >> 4)) * 256 + (j & 15) * 16 + (i & 15);
    const double s = red[0][e] + red[1][e] + red[2][e] + red[3][e];
    if (P.nb > 1) {
      P.part[((int64_t)bi * P.nb + g) * nout + o] = s;
    } else {
      double* c = P.C + bi * P.sc + i + P.ldc * j;
      *c = P.alpha * s + (P.beta == 0.0 ? 0.0 : P.beta * *c);
    }
  }
}

// A wave per entry; with few slices (WAVE false) a thread: 368640 entries of two took 77 us
// with a wave each.
template <bool WAVE>
__global__ __launch_bounds__(256) void k_tn_sum(const TnArgs P) {
  if constexpr (!WAVE) {
    const int nout = P.M * P.N;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)nout * P.nbatch) return;
    const int bi = (int)(t / nout), o = (int)(t % nout);
    const double* part = P.part + (int64_t)bi * P.nb * nout + o;
    double s = 0.0;
#pragma unroll 8
    for (int g = 0; g < P.nb; ++g) s += part[(int64_t)g * nout];
    double* c = P.C + bi * P.sc + (o % P.M) + P.ldc * (o / P.M);
    *c = P.alpha * s + (P.beta == 0.0 ? 0.0 : P.beta * *c);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t ow = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int nout = P.M * P.N;
  if (ow >= (int64_t)nout * P.nbatch) return;
  const int bi = (int)(ow / nout), o = (int)(ow % nout);
  const double* part = P.part + (int64_t)bi * P.nb * nout;
  double s = 0.0;
  for (int g = lane; g < P.nb; g += 64) s += part[(int64_t)g * nout + o];
  s = wsum(s);
  if (lane == 0) {
    double* c = P.C + bi * P.sc + (o % P.M) + P.ldc * (o / P.M);
    *c = P.alpha * s + (P.beta == 0.0 ? 0.0 : P.beta * *c);
  }
}

template <bool PAIR>
void launch_tn(TnArgs P, hipStream_t s) {
  const int64_t blocks = (int64_t)P.nb * P.nbatch;
  const dim3 b(256);
  for (P.blk0 = 0; P.blk0 < blocks; P.blk0 += kMaxGrid) {
    const dim3 g((unsigned)std::min(blocks - P.blk0, kMaxGrid));
    if (P.M <= 16 && P.N <= 16) hipLaunchKernelGGL((k_tn<1, 1, PAIR>), g, b, 0, s, P);
    else if (P.M <= 16) hipLaunchKernelGGL((k_tn<1, 2, PAIR>), g, b, 0, s, P);
    else if (P.N <= 16) hipLaunchKernelGGL((k_tn<2, 1, PAIR>), g, b, 0, s, P);
    else hipLaunchKernelGGL((k_tn<2, 2, PAIR>), g, b, 0, s, P);
  }
}

hipError_t run_tn(TnArgs P, hipStream_t s) {
  if (P.M <= 0 || P.N <= 0 || P.nbatch <= 0) return hipSuccess;
  if (P.M > PSTT2_MAX_ELL || P.N > PSTT2_MAX_ELL || P.K < 1) return hipErrorInvalidValue;
  // slices of 128 rows (a wave's four steps) and longer while about 1024
  // workgroups remain: the partials, 8 M N bytes a slice, are written and read back
  int64_t rows = 128;
  while (rows < 4096 && (P.K + 2 * rows - 1) / (2 * rows) * P.nbatch >= 1024) rows *= 2;
  // whole where that leaves two workgroups to a compute unit: no partials (960 products
  // of K = 960, 12 x 32: 127 us with two slices each, 45 whole)
  if (P.K <= 2 * rows && P.nbatch >= 512) rows = (P.K + 31) / 32 * 32;
  P.rows = rows;
  P.nb = (int)((P.K + rows - 1) / rows);
  P.part = nullptr;
  if (P.nb > 1) {
    const hipError_t e = ws_alloc((void**)&P.part, sizeof(double) * P.nb * P.nbatch * P.M * P.N, s);
    if (e != hipSuccess) return e;
  }
  // 16-byte loads: contiguous rows, even strides and counts, aligned operands
  const bool pair = P.ra == 1 && P.rb == 1 && ((P.lda | P.ldb | P.sa | P.sb | P.K) & 1) == 0 &&
                    (((uintptr_t)P.A | (uintptr_t)P.B) & 15) == 0;
  if (pair) launch_tn<true>(P, s);
  else launch_tn<false>(P, s);
  if (P.nb > 1) {
    const int64_t out = (int64_t)P.M * P.N * P.nbatch;
    if (P.nb > 16) hipLaunchKernelGGL(k_tn_sum<true>, dim3((unsigned)((out + 3) / 4)), dim3(256), 0, s, P);
    else hipLaunchKernelGGL(k_tn_sum<false>, dim3((unsigned)((out + 255) / 256)), dim3(256), 0, s, P);
    ws_free(P.part, s);
  }
  return hipGetLastError();
}

}  // namespace

// op(B)(k, j): B is K x N (tb false) or N x K (tb true); at(B, ldb, !tb, j, k) reads it.
hipError_t adj_gemm(bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha, const double* A, int64_t lda,
                    const double* B, int64_t ldb, double beta, double* C, int64_t ldc, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (ta && !tb && M <= 32 && N <= 32 && K >= 256)
    return run_tn(TnArgs{(int)M, (int)N, K, A, lda, 1, 0, B, ldb, 1, 0, alpha, beta, C, ldc, 0, 1, 0, 0, nullptr, 0}, s);
  const int64_t tiles = (M + 15) / 16 * ((N + 15) / 16);
  // long contractions with few outputs spread over one wavefront per entry
  if (K >= 256 && M * N <= 65536)
    hipLaunchKernelGGL(k_gemm_w, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((M * N + 3) / 4, 16384))),
                       dim3(256), 0, s, ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
  else {
    const bool split = K >= 32;
    const int64_t blocks = split ? tiles : (tiles + 3) / 4;
    for (int64_t b0 = 0; b0 < blocks; b0 += kMaxGrid) {
      const dim3 g((unsigned)std::min(blocks - b0, kMaxGrid));
      if (split)
        hipLaunchKernelGGL(k_gemm_m<true>, g, dim3(256), 0, s, ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, b0);
      else
        hipLaunchKernelGGL(k_gemm_m<false>, g, dim3(256), 0, s, ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, b0);
    }
  }
  return hipGetLastError();
}

hipError_t adj_gemm_tn_batch(int64_t M, int64_t N, int64_t K, int nbatch, const double* A, int64_t lda, int64_t ra,
                             int64_t sa, const double* B, int64_t ldb, int64_t sb, double* C, int64_t ldc, int64_t sc,
                             hipStream_t s) {
  return run_tn(TnArgs{(int)M, (int)N, K, A, lda, ra, sa, B, ldb, 1, sb, 1.0, 0.0, C, ldc, sc, nbatch, 0, 0, nullptr, 0},
                s);
}

}  // namespace pstt2
