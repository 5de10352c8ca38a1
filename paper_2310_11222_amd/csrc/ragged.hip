// Laplacian apply Y = L X on a number of columns that is no power of two, in
// one pass over the graph: the plain apply (k_spmm) runs such an X as a pass
// for every power of two in it, and on a large graph every pass costs the
// same requests for the neighbours' rows whatever their width.
//
// A row of X is read by the next power of two of lanes, one element a lane
// (rows of 3 or 5 elements have no 16-byte alignment to use); the lanes past
// the last column repeat it, so that they ask for no further line, and store
// nothing.  Rows and the split of long rows are those of k_spmm.
//
// FP32 sums are those of k_spmm, in its order, but for two kinds that are FP64
// sums rounded once: of long rows, of which a lane per element takes up to four
// times as many terms as k_spmm's lanes (in FP32 hubs were 2.4 times as far from
// the exact values), and (SpmmCall::wide) of every row where the odd column had the
// sums of the sliced apply before it came into this pass.
//
// Measured (us, a pass for every power of two -> one pass): power law n = 10^6
// weighted, FP32 3 columns 230 -> 155, 7 columns 419 -> 203, 15 columns 667 -> 278
// (all sums in FP64 159, 209 and 291), FP64 13 columns 609 -> 333; BA n = 3,000,
// 13 columns 37 -> 16.
#include <algorithm>

#include "device_common.hpp"
#include "prof.hpp"

namespace nvd {

template <typename V>
struct RaggedK {
  int n, cols;
  const int* rp;
  const int* ci;
  const V* w;
  const V* x;
  long ldx;
  V* y;
  long ldy;
  int nlong_blocks;
};

// A: the type of the short rows' sums.
template <typename V, typename A, int L, bool UNIT>
__global__ __launch_bounds__(kBS) void k_apply_ragged(RaggedK<V> a, LongRows lr) {
  __shared__ double sh[kBS];
  __shared__ int s_last;
  const int t = threadIdx.x;
  const int c = t % L;
  const int cc = min(c, a.cols - 1);
  if ((int)blockIdx.x < a.nlong_blocks) {
    // a segment of a long row: L lanes by 256 / L neighbours
    constexpr int NJ = kBS / L;
    for (int s = blockIdx.x; s < lr.n_seg; s += a.nlong_blocks) {
      const int row = lr.seg_row[s];
      const int hi = lr.seg_hi[s];
      const double own = (double)a.x[(long)row * a.ldx + cc];
      double sum = 0.0;
      for (int e = lr.seg_lo[s] + t / L; e < hi; e += NJ)
        sum += (UNIT ? 1.0 : (double)a.w[e]) * (own - (double)a.x[(long)a.ci[e] * a.ldx + cc]);
      const double part[1][1] = {{sum}};
      block_reduce_cols<kBS, 1, 1>(part, L, sh);
      const int first = lr.seg_first[s], cnt = lr.seg_cnt[s];
      if (cnt == 1) {
        if (t < a.cols) a.y[(long)row * a.ldy + t] = (V)sh[t];
      } else {
        if (t < L) st_agent(&lr.seg_part[(long)s * kMaxTile + t], sh[t]);
        wait_stores();
        __syncthreads();
        if (t == 0) s_last = (ticket(&lr.row_tick[first]) == (unsigned)(cnt - 1));
        __syncthreads();
        if (s_last) {
          if (t < a.cols) {
            double all = 0.0;
            for (int i = 0; i < cnt; ++i) all += ld_agent(&lr.seg_part[(long)(first + i) * kMaxTile + t]);
            a.y[(long)row * a.ldy + t] = (V)all;
          }
          if (t == 0) lr.row_tick[first] = 0u;
        }
      }
      __syncthreads();
    }
    return;
  }
  // short rows: a lane group per row, eight neighbours a step
  constexpr int U = 8;
  constexpr int RB = kBS / L;      // rows of a block's step
  const int nsb = gridDim.x - a.nlong_blocks;
  for (long row = (long)((int)blockIdx.x - a.nlong_blocks) * RB + t / L; row < a.n; row += (long)nsb * RB) {
    const int lo = a.rp[row];
    const int deg = a.rp[row + 1] - lo;
    if (deg > kLongRow) continue;
    const A own = (A)a.x[row * a.ldx + cc];
    A sum = (A)0;
    for (int e0 = 0; e0 < deg; e0 += U) {
      int col[U];
      V wt[U], xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = e0 + u < deg;
        col[u] = in ? a.ci[lo + e0 + u] : 0;
        wt[u] = in ? (UNIT ? (V)1 : a.w[lo + e0 + u]) : (V)0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) xv[u] = e0 + u < deg ? a.x[(long)col[u] * a.ldx + cc] : (V)0;
      if constexpr (sizeof(A) != sizeof(V)) {
        // all loads are out before the first conversion: it would otherwise move
        // up behind each load's own test and wait for it there
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" : "+v"(wt[u]), "+v"(xv[u]));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) sum += (A)wt[u] * (own - (A)xv[u]);
    }
    if (c < a.cols) __builtin_nontemporal_store((V)sum, &a.y[row * a.ldy + c]);
  }
}

template <typename V, typename A>
static nvd_status launch_ragged_t(const SpmmCall& c, int cols, hipStream_t s) {
  const DevGraph* g = c.g;
  RaggedK<V> k{};
  k.n = g->n;
  k.cols = cols;
  k.rp = g->rp;
  k.ci = g->ci;
  const bool unit = !g->weighted;
  k.w = sizeof(V) == 8 ? (const V*)g->w64 : (const V*)g->w32;
  k.x = static_cast<const V*>(c.x);
  k.ldx = c.ldx;
  k.y = static_cast<V*>(c.y);
  k.ldy = c.ldy;
  k.nlong_blocks = std::min(g->lr.n_seg, 1024);
  const int rows = kBS / c.T;
  const long steps = ((long)g->n + rows - 1) / rows;
  const int grid = k.nlong_blocks + (int)std::max<long>(1, std::min<long>(steps, kMaxBlocks - 1024));
  int pid = -1;
  if (prof_enabled()) {
    const double sv = (double)sizeof(V), sw = unit ? 0.0 : sv, n = g->n;
    pid = prof_begin(s, sizeof(V) == 8 ? PK_SPMM64 : PK_SPMM32,
                     (4.0 + sw) * g->nnz + 4.0 * (n + 1) + 2.0 * cols * sv * n);
  }
  switch (c.T) {
#define NVD_R(LL)                                                        \
  case LL:                                                               \
    if (unit)                                                            \
      k_apply_ragged<V, A, LL, true><<<grid, kBS, 0, s>>>(k, g->lr);        \
    else                                                                 \
      k_apply_ragged<V, A, LL, false><<<grid, kBS, 0, s>>>(k, g->lr);       \
    break;
    NVD_R(4) NVD_R(8) NVD_R(16) NVD_R(32) NVD_R(64)
#undef NVD_R
    default: break;
  }
  prof_end(s, pid);
  NVD_HIP(hipGetLastError());
  return NVD_OK;
}

nvd_status launch_ragged(const SpmmCall& c, int cols, hipStream_t s) {
  if (c.prec == 0) return launch_ragged_t<double, double>(c, cols, s);
  return c.wide ? launch_ragged_t<float, double>(c, cols, s) : launch_ragged_t<float, float>(c, cols, s);
}

}  // namespace nvd
