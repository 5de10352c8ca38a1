// Work by CSR entry: checking new edge weights and the adjoint for the weights;
// and weighted degrees, sixteen lanes a row.
//
// A thread (or lane group) per row left the first two as long as their longest
// row, and the degrees sixteen times as long as they are now: on a BA graph of 2 10^5 nodes (m = 5, hubs of thousands) the check took
// 5.5 ms, the degrees 0.42 and the adjoint over 32 columns 1.9, of a training
// step of 20.  By entry they need an entry's row and the place of its mirror
// entry; both are found when weights are first replaced, by bisection, and kept
// (8 bytes an entry; without the memory for them they are found in each call).
// That step then took 12.3 ms.
#include <algorithm>

#include "column_pre_dev.hpp"
#include "entry_walk.hpp"

namespace nvd {

// Row of entry e: the last one that starts at or before it.
__device__ __forceinline__ int row_of(int n, const int* __restrict__ rp, int e) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = lo + (hi - lo) / 2;
    if (rp[mid] <= e)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The entry (j, i) of an entry (i, j) (the graph was checked to be symmetric).
__device__ __forceinline__ int mirror_of(const int* __restrict__ rp, const int* __restrict__ ci, int i, int j) {
  int a = rp[j], b = rp[j + 1];
  while (a < b) {
    const int mid = a + (b - a) / 2;
    if (ci[mid] < i)
      a = mid + 1;
    else
      b = mid;
  }
  return a;
}

// Row and mirror entry of every entry.
__global__ __launch_bounds__(kEntryBS) void k_entries(int n, int nnz, const int* __restrict__ rp,
                                                      const int* __restrict__ ci, int* __restrict__ erow,
                                                      int* __restrict__ mirror) {
  for_entries(blockIdx.x, gridDim.x, threadIdx.x, nnz, [&](int e) {
    const int i = row_of(n, rp, e);
    erow[e] = i;
    mirror[e] = mirror_of(rp, ci, i, ci[e]);
  });
}

// New weights in input order: bit 1 where one is not finite and positive, bit 2
// where an entry's and its mirror's differ.  mirror may be null.
__global__ __launch_bounds__(kEntryBS) void k_check_entries(int n, int nnz, const int* __restrict__ rp,
                                                            const int* __restrict__ ci,
                                                            const int* __restrict__ in_pos,
                                                            const int* __restrict__ mirror,
                                                            const double* __restrict__ w, int* flag) {
  int bad = 0;
  for_entries(blockIdx.x, gridDim.x, threadIdx.x, nnz, [&](int e) {
    const int m = mirror ? mirror[e] : mirror_of(rp, ci, row_of(n, rp, e), ci[e]);
    const double v = w[in_pos ? in_pos[e] : e];
    if (!(v > 0.0) || !isfinite(v)) bad |= 1;
    if (w[in_pos ? in_pos[m] : m] != v) bad |= 2;
  });
  if (bad) atomicOr(flag, bad);
}

// Weighted degrees and their inverses (w64 null: unit weights), sixteen lanes a
// row; w32, where given, receives the weights in FP32.
__global__ __launch_bounds__(256) void k_row_degree(int n, const int* __restrict__ rp,
                                                    const double* __restrict__ w64, float* __restrict__ w32,
                                                    double* __restrict__ deg64, float* __restrict__ deg32,
                                                    double* __restrict__ invd64, float* __restrict__ invd32) {
  const int lane = threadIdx.x & 15;
  for (long i = (long)blockIdx.x * 16 + (threadIdx.x >> 4); i < n; i += (long)gridDim.x * 16) {
    const int lo = rp[i], hi = rp[i + 1];
    double d = 0.0;
    if (w64) {
      for (int e = lo + lane; e < hi; e += 16) {
        const double w = w64[e];
        d += w;
        if (w32) w32[e] = (float)w;
      }
      d = row16_sum(d);
    } else {
      d = (double)(hi - lo);
    }
    if (lane == 0) {
      deg64[i] = d;
      deg32[i] = (float)d;
      const double inv = d > 0.0 ? 1.0 / d : 0.0;
      invd64[i] = inv;
      invd32[i] = (float)inv;
    }
  }
}

// gw[e] = -1/2 sum_c g_c (X[i, c] - X[j, c])^2 over `cols` <= L columns: L lanes
// an entry, four entries in flight a group (of one row, mostly: its X is read
// from L1 after the first).  erow may be null: the rows are then found here
// (the call allocates nothing, so that it can be captured at any time).
template <int L>
__global__ __launch_bounds__(256) void k_grad_entries(int n, int nnz, const int* __restrict__ rp,
                                                      const int* __restrict__ erow,
                                                      const int* __restrict__ ci,
                                                      const int* __restrict__ in_pos,
                                                      const double* __restrict__ X, long ldx,
                                                      const double* __restrict__ gs, int cols,
                                                      double* __restrict__ gw, int accumulate) {
  constexpr int U = 4;
  constexpr int LOG = L == 1 ? 0 : L == 2 ? 1 : L == 4 ? 2 : L == 8 ? 3 : L == 16 ? 4 : L == 32 ? 5 : 6;
  const int c = threadIdx.x % L;
  const int cc = min(c, cols - 1);
  const double gc = -0.5 * gs[cc];
  const long groups = (long)gridDim.x * (256 / L);
  for (long q = (long)blockIdx.x * (256 / L) + threadIdx.x / L; q * U < nnz; q += groups) {
    const int e0 = (int)(q * U);
    int row[U];
    if (erow) {
#pragma unroll
      for (int u = 0; u < U; ++u) row[u] = erow[min(e0 + u, nnz - 1)];
    } else {
      row[0] = row_of(n, rp, e0);
#pragma unroll
      for (int u = 1; u < U; ++u) {
        row[u] = row[u - 1];
        while (rp[row[u] + 1] <= min(e0 + u, nnz - 1)) ++row[u];
      }
    }
    double df[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = min(e0 + u, nnz - 1);
      df[u] = X[(long)row[u] * ldx + cc] - X[(long)ci[e] * ldx + cc];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (nothing of the lanes past the last column, whatever X holds there)
      const double v = group_sum(c < cols ? gc * df[u] * df[u] : 0.0, LOG);
      if (c == 0 && e0 + u < nnz) {
        const long pos = in_pos ? in_pos[e0 + u] : e0 + u;
        gw[pos] = accumulate ? gw[pos] + v : v;
      }
    }
  }
}

void launch_row_degree(int n, const int* rp, const double* w64, float* w32, double* deg64, float* deg32,
                       double* invd64, float* invd32, hipStream_t s) {
  k_row_degree<<<entry_grid(16L * n), 256, 0, s>>>(n, rp, w64, w32, deg64, deg32, invd64, invd32);
}

static nvd_status ensure_entries(DevGraph* g, hipStream_t s) {
  if (g->erow) return NVD_OK;
  int* p = nullptr;
  const size_t count = 2 * (size_t)std::max(g->nnz, 1) + 1;
  NVD_HIP(device_alloc((void**)&p, sizeof(int) * count));
  if (g->nnz > 0) k_entries<<<entry_grid(g->nnz), kEntryBS, 0, s>>>(g->n, g->nnz, g->rp, g->ci, p, p + g->nnz);
  // (other streams may use them from the next call on)
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    (void)hipFree(p);
    set_error(std::string("entries: ") + hipGetErrorString(e));
    return NVD_E_DEVICE;
  }
  g->erow = p;
  g->mirror = p + g->nnz;
  g->bytes += (int64_t)(sizeof(int) * count);
  return NVD_OK;
}

// Bits of k_check_entries for the new weights w (input order); waits for s.
nvd_status check_weights(DevGraph* g, const double* w, int* bits, hipStream_t s) {
  const nvd_status st = ensure_entries(g, s);
  if (st != NVD_OK && st != NVD_E_NOMEM) return st;
  int* own = nullptr;              // the word of a call without the map
  if (st == NVD_E_NOMEM) {
    set_error("");
    NVD_HIP(device_alloc((void**)&own, sizeof(int)));
  }
  int* flag = own ? own : g->erow + 2 * (size_t)std::max(g->nnz, 1);
  *bits = 0;
  hipError_t e = hipMemcpyAsync(flag, bits, sizeof(int), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && g->nnz > 0) {
    k_check_entries<<<std::min(entry_grid(g->nnz), 2048), kEntryBS, 0, s>>>(g->n, g->nnz, g->rp, g->ci, g->in_pos,
                                                                            g->mirror, w, flag);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(bits, flag, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(own);
  NVD_HIP(e);
  return NVD_OK;
}

nvd_status grad_entries(DevGraph* g, int k, const double* X, int64_t ldx, const double* gs, double* gw,
                        hipStream_t s) {
  if (g->nnz == 0) return NVD_OK;
  for (int c0 = 0; c0 < k; c0 += 64) {
    const int cols = std::min(64, k - c0);
    int L = 1;
    while (L < cols) L *= 2;
    const int grid = entry_grid(((long)g->nnz + 3) / 4 * L);
    switch (L) {
#define NVD_E(LL)                                                                                          \
  case LL:                                                                                                 \
    k_grad_entries<LL><<<grid, 256, 0, s>>>(g->n, g->nnz, g->rp, g->erow, g->ci, g->in_pos, X + c0, ldx,   \
                                            gs + c0, cols, gw, c0 > 0 ? 1 : 0);                                                      \
    break;
      NVD_E(1) NVD_E(2) NVD_E(4) NVD_E(8) NVD_E(16) NVD_E(32) NVD_E(64)
#undef NVD_E
      default: break;
    }
    NVD_HIP(hipGetLastError());
  }
  return NVD_OK;
}

// The host's copy of the weights, where they were replaced since it was taken.
nvd_status ensure_host_weights(DevGraph* g) {
  if (!g->h_w_stale) return NVD_OK;
  g->h_w.resize(g->nnz);
  if (g->nnz > 0)
    NVD_HIP(hipMemcpy(g->h_w.data(), g->w64, sizeof(double) * g->nnz, hipMemcpyDeviceToHost));
  g->h_w_stale = false;
  return NVD_OK;
}

}  // namespace nvd
