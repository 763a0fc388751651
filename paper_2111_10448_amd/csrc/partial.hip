// Partial columns: slab edges that cut a column of the pass's unfolding X_m.
// Every entry of a piece enters both sketches in FP64, whatever the sketch
// precision,
//     Y_R(r, :) += x(r) Omega_m(col, :),   T_m(:, col) += sum_r Psi_m(r, :) x(r).
#include <algorithm>

#include "drm.h"

namespace pstt2 {

typedef double pc_d4 __attribute__((ext_vector_type(4)));

constexpr int PC_ROWS = 256;        // rows of X_m per workgroup step (64 per wave)
constexpr int PC_MAXBLK = 1024;     // workgroups per launch at most

// The pieces of a call are the columns of a narrow matrix (zero outside each
// piece's rows), so 16 of them at a time go through the dual product on FP64
// matrix cores, as a 16-column chunk does in the streaming kernel: a wave
// stages its 64 rows x 16 pieces in LDS and
//     Y(rows, ell) += X(rows, 16 pieces) Omega(piece columns, ell)
//     T(ell, 16 pieces) = Psi(rows, ell)^T X(rows, pieces).
// A workgroup owns 256 rows of Y_R and walks the chunks with a piece in them, so Y is
// read and written once per launch with one writer per entry; T goes to one
// partial per workgroup, summed in a fixed order by k_partial_t.  The work list
// holds the row blocks that some piece touches and no others, since a call may
// bring one fibre of a very tall unfolding (walking all of Y_R for it took 5.4 ms
// a call at R = 2^25, ell = 20; now 22 us).  Workgroups step over the list when it
// has more than PC_MAXBLK blocks.
// Latency bound: one launch pair per kMaxSeg pieces, against a single
// workgroup per piece before (0.42-0.44 ms each at R = 19575, ell = 20 and
// R = 20592, ell = 16).  A half-precision pass over 3.5e8 entries in 64 slabs
// with 112 such pieces: 52.7 -> 3.35 ms; an FP64 pass over 1.2e7 entries in 9
// slabs with per-split factors (3 x 16 pieces): 21.4 -> 0.68 ms.
// Pieces: seg[e].ptr the first entry, gcol0 the column, rows [chunk0, ncols).
struct RowBlocks {
  int n;                     // runs of consecutive row blocks, increasing and disjoint
  int64_t tot;               // blocks in all
  int64_t first[kMaxSeg];    // first block of each run
  int64_t before[kMaxSeg];   // blocks of the runs before it
};

template <int L4, typename T>
__global__ __launch_bounds__(256, 2) void k_partial_cols(const SketchArgs A, const RowBlocks B, double* __restrict__ Y,
                                                         double* __restrict__ tws) {
  constexpr int ST = 64 + 2;
  constexpr int NQ = L4 / 16;        // 16-wide tiles of the sketch columns
  constexpr int NS = (L4 % 16) / 4;  // 4-wide groups
  constexpr int KT = 16;             // K steps over a wave's rows
  __shared__ double Xl[4][16 * ST];
  __shared__ double Tred[4][L4 * 16];
  __shared__ double Tsum[kMaxSeg / 16][L4 * 16];
  __shared__ const T* ep[kMaxSeg];
  __shared__ int64_t e0[kMaxSeg], e1[kMaxSeg], ec[kMaxSeg];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int l16 = lane & 15, g4 = lane >> 4, l4 = lane & 3, blk = (lane >> 2) & 3;
  const int ne = A.nseg;
  const int nch = (ne + 15) / 16;
  // pieces past the last one: no rows, column 0
  if (t < kMaxSeg) {
    const bool in = t < ne;
    ep[t] = in ? (const T*)A.seg[in ? t : 0].ptr : nullptr;
    e0[t] = in ? A.seg[in ? t : 0].chunk0 : 0;
    e1[t] = in ? A.seg[in ? t : 0].ncols : 0;
    ec[t] = in ? A.seg[in ? t : 0].gcol0 : 0;
  }
  for (int i = t; i < nch * L4 * 16; i += 256) (&Tsum[0][0])[i] = 0.0;
  __syncthreads();   // the piece table
  for (int64_t i = blockIdx.x; i < B.tot; i += gridDim.x) {
    int run = 0;
    while (run + 1 < B.n && B.before[run + 1] <= i) ++run;
    const int64_t rb = B.first[run] + (i - B.before[run]);
    // pieces with rows in this block, the same mask in every wave
    const uint64_t here = __ballot(lane < ne && e0[lane < kMaxSeg ? lane : 0] < (rb + 1) * PC_ROWS &&
                                   e1[lane < kMaxSeg ? lane : 0] > rb * PC_ROWS);
    const int64_t row0w = rb * PC_ROWS + w * 64;
    double psiq[KT][NQ > 0 ? NQ : 1];
    double psis[KT][NS > 0 ? NS : 1];
    {
      int cols[NQ + NS];
#pragma unroll
      for (int q = 0; q < NQ; ++q) cols[q] = 16 * q + l16;
#pragma unroll
      for (int s = 0; s < NS; ++s) cols[NQ + s] = 16 * NQ + 4 * s + l4;
      auto fill = [&](auto rows) {
        rows.init(A, row0w + g4);
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) {
          double v[NQ + NS];
          if (ks > 0) rows.advance(A, 4);
          rows.values(A, cols, v);
#pragma unroll
          for (int q = 0; q < NQ; ++q) psiq[ks][q] = v[q];
#pragma unroll
          for (int s = 0; s < NS; ++s) psis[ks][s] = v[NQ + s];
        }
      };
      static_assert(psi_stage_size(PC_ROWS, L4) <= 4 * 16 * ST, "the table fits in the X tiles");
      __syncthreads();   // the last row block's reads of them are done
      if (A.psi_tab) fill(PsiTable<NQ + NS>(A));
      else if (psi_stage(A, rb * PC_ROWS, PC_ROWS, &Xl[0][0])) fill(PsiStaged<NQ + NS>(A, &Xl[0][0], rb * PC_ROWS));
      else fill(PsiDirect<NQ + NS>());
    }
    pc_d4 yq[4][NQ > 0 ? NQ : 1];
    double ys[4][NS > 0 ? NS : 1];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) yq[mt][q] = pc_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < NS; ++s) ys[mt][s] = 0.0;
    }
    for (int ch = 0; ch < nch; ++ch) {
      if ((here >> (16 * ch) & 0xffff) == 0) continue;   // uniform across the workgroup
      __syncthreads();   // the last chunk's LDS reads are done
      const int64_t row = row0w + lane;
      double v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int e = 16 * ch + j;
        v[j] = (row >= e0[e] && row < e1[e]) ? (double)ep[e][row - e0[e]] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) Xl[w][j * ST + lane] = v[j];
      __syncthreads();
      const double* xw = Xl[w];
      pc_d4 tq[NQ > 0 ? NQ : 1];
      double ts[NS > 0 ? NS : 1];
#pragma unroll
      for (int q = 0; q < NQ; ++q) tq[q] = pc_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < NS; ++s) ts[s] = 0.0;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int col = 4 * ks + g4;
        const double* om = A.om_tab + ec[16 * ch + col] * A.L4;
        double bq[NQ > 0 ? NQ : 1], bs[NS > 0 ? NS : 1];
#pragma unroll
        for (int q = 0; q < NQ; ++q) bq[q] = om[16 * q + l16];
#pragma unroll
        for (int s = 0; s < NS; ++s) bs[s] = om[16 * NQ + 4 * s + l4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const double a = xw[col * ST + 16 * mt + l16];
#pragma unroll
          for (int q = 0; q < NQ; ++q) yq[mt][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bq[q], yq[mt][q], 0, 0, 0);
#pragma unroll
          for (int s = 0; s < NS; ++s) ys[mt][s] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, bs[s], ys[mt][s], 0, 0, 0);
        }
      }
#pragma unroll
      for (int ks = 0; ks < KT; ++ks) {
        const double b = xw[l16 * ST + 4 * ks + g4];
#pragma unroll
        for (int q = 0; q < NQ; ++q) tq[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(psiq[ks][q], b, tq[q], 0, 0, 0);
#pragma unroll
        for (int s = 0; s < NS; ++s) ts[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(psis[ks][s], b, ts[s], 0, 0, 0);
      }
      double* tr = Tred[w];
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) tr[(16 * q + 4 * u + g4) * 16 + l16] = tq[q][u];
#pragma unroll
      for (int s = 0; s < NS; ++s) tr[(16 * NQ + 4 * s + g4) * 16 + 4 * blk + l4] = ts[s];
      __syncthreads();
      // each thread owns its entries of the running sum
      for (int i = t; i < L4 * 16; i += 256) Tsum[ch][i] += Tred[0][i] + Tred[1][i] + Tred[2][i] + Tred[3][i];
    }
    auto put = [&](int64_t row, int c, double v) {
      if (row < A.R && c < A.ell) Y[(int64_t)c * A.R + row] += v;
    };
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) put(row0w + 16 * mt + 4 * u + g4, 16 * q + l16, yq[mt][q][u]);
#pragma unroll
      for (int s = 0; s < NS; ++s) put(row0w + 16 * mt + 4 * blk + g4, 16 * NQ + 4 * s + l4, ys[mt][s]);
    }
  }
  __syncthreads();
  // partial [workgroup][piece][a]
  for (int i = t; i < ne * L4; i += 256) {
    const int e = i / L4, a = i % L4;
    tws[((int64_t)blockIdx.x * ne + e) * L4 + a] = Tsum[e / 16][a * 16 + e % 16];
  }
}

// T_m(a, col) += the piece's partials, one wavefront per (piece, a): lanes take
// workgroups lane, lane + 64, ... and a fixed butterfly adds them.  Pieces of one
// column (a slab's tail and the next one's head) are added in launch order by
// the first one's wavefront.
__global__ __launch_bounds__(256) void k_partial_t(const SketchArgs A, const double* __restrict__ tws, int nb, int L4,
                                                   double* __restrict__ Tt) {
  const int lane = threadIdx.x & 63;
  const int o = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
  if (o >= A.nseg * A.ell) return;
  const int e = o / A.ell, a = o % A.ell;
  const int64_t col = A.seg[e].gcol0;
  for (int k = 0; k < e; ++k)
    if (A.seg[k].gcol0 == col) return;   // uniform across the wavefront
  double s = Tt[(int64_t)a * A.C + col];
  for (int k = e; k < A.nseg; ++k) {
    if (A.seg[k].gcol0 != col) continue;
    double p = 0.0;
    for (int g = lane; g < nb; g += 64) p += tws[((int64_t)g * A.nseg + k) * L4 + a];
    for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off);
    s += p;
  }
  if (lane == 0) Tt[(int64_t)a * A.C + col] = s;
}

template <typename T>
static void launch_pc(int L4, const SketchArgs& a, const RowBlocks& rb, int nb, double* Y, double* tws, hipStream_t s) {
  const dim3 g((unsigned)nb), b(256);
  switch (L4) {
    case 4: hipLaunchKernelGGL((k_partial_cols<4, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 8: hipLaunchKernelGGL((k_partial_cols<8, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 12: hipLaunchKernelGGL((k_partial_cols<12, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 16: hipLaunchKernelGGL((k_partial_cols<16, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 20: hipLaunchKernelGGL((k_partial_cols<20, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 24: hipLaunchKernelGGL((k_partial_cols<24, T>), g, b, 0, s, a, rb, Y, tws); break;
    case 28: hipLaunchKernelGGL((k_partial_cols<28, T>), g, b, 0, s, a, rb, Y, tws); break;
    default: hipLaunchKernelGGL((k_partial_cols<32, T>), g, b, 0, s, a, rb, Y, tws); break;
  }
}

int64_t partial_cols_doubles(int64_t R, int L4, int pieces) {
  return std::min<int64_t>((R + PC_ROWS - 1) / PC_ROWS, PC_MAXBLK) * pieces * L4;
}

// The row blocks that the pieces touch.
static RowBlocks touched_blocks(const SketchArgs& a) {
  int64_t lo[kMaxSeg], hi[kMaxSeg];
  int order[kMaxSeg];
  for (int e = 0; e < a.nseg; ++e) {
    lo[e] = a.seg[e].chunk0 / PC_ROWS;
    hi[e] = (a.seg[e].ncols + PC_ROWS - 1) / PC_ROWS;
    order[e] = e;
  }
  std::sort(order, order + a.nseg, [&](int p, int q) { return lo[p] < lo[q]; });
  RowBlocks b = {};
  int64_t end = 0;   // blocks before it are listed
  for (int i = 0; i < a.nseg; ++i) {
    const int64_t from = std::max(lo[order[i]], end), to = hi[order[i]];
    if (from >= to) continue;
    if (b.n == 0 || from > end) {
      b.first[b.n] = from;
      b.before[b.n++] = b.tot;
    }
    b.tot += to - from;
    end = to;
  }
  return b;
}

hipError_t launch_partial_cols(int dtype, const SketchArgs& a, double* Y, double* Tt, double* ws, int64_t ws_doubles,
                               bool* added, hipStream_t s) {
  if (a.nseg < 1 || a.nseg > kMaxSeg || a.ell < 1 || a.L4 < a.ell || a.L4 % 4 != 0 || a.L4 > 32) return hipErrorInvalidValue;
  const RowBlocks rb = touched_blocks(a);
  const int64_t per = (int64_t)a.nseg * a.L4;
  const int nb = (int)std::min<int64_t>({rb.tot, (int64_t)PC_MAXBLK, ws_doubles / per});
  if (nb < 1) return hipErrorInvalidValue;
  if (fault_take()) return hipErrorLaunchFailure;
  if (dtype == PSTT2_F64) launch_pc<double>(a.L4, a, rb, nb, Y, ws, s);
  else launch_pc<float>(a.L4, a, rb, nb, Y, ws, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  *added = true;
  hipLaunchKernelGGL(k_partial_t, dim3((unsigned)((a.nseg * a.ell + 3) / 4)), dim3(256), 0, s, a, ws, nb, a.L4, Tt);
  return hipGetLastError();
}

}  // namespace pstt2
