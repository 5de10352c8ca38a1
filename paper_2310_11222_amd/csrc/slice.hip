// Laplacian apply of one right-hand-side column (T = 1) on large graphs, by
// column slices held in LDS.  Same operator as k_spmm (the paper's
// section 3.1 L = D - A):
//   (L x)_v = sum_u w_vu (x_v - x_u).
//
// On a large random graph a one-column apply is bound by its neighbour
// gathers: each reads 4 or 8 bytes of x and brings a 128-byte line from
// beyond the XCD's 4 MB L2, and even gathers that hit the L2 are bound by its
// rate of requests (the form that held slices of x in the L2s and wrote one
// partial sum per row and slice ran at 0.69 ms per FP32 apply, about 1.3 TB/s
// of its traffic, on the 10^7-node graph below).  LDS answers random reads an
// order of magnitude faster, so here the gathers are made there and everything
// else is a stream.  The columns (nodes) are cut into slices of kSlNodes, and
// the rows into chunks of consecutive rows with at most kSlChunk CSR entries:
//  * gather: the entries, ordered by (slice, chunk, CSR position), are split
//    evenly over the blocks.  A block loads the slice of x that its entries
//    lie in into LDS, reads the entries' 2-byte columns within the slice and
//    writes the neighbours' values x_u in the same order.  An even split of
//    the entries needs no balance between slices: a block that crosses into
//    the next slice loads that one too.
//  * rows: a block per chunk at a time.  The chunk's values lie in one run per
//    slice; L lanes take a run, and put its values at their 2-byte positions,
//    the entries' CSR order within the chunk, in LDS.  Then a thread per
//    row sums w_vu (x_v - x_u) in FP64 in CSR order, with the weights read
//    from the graph's own CSR (rows of more than kSlGroupRow entries
//    are summed by 16 lanes, of more than kSlWaveRow by the wave), rounds once, and does the epilogue of the apply
//    (store, CG dot p^T q, or the FP64 residual r = b - L x and its dots) as
//    in k_spmm.  Neighbouring chunks, whose runs share lines, go to blocks of
//    one XCD.
// A row of more than kSlChunk entries is a chunk of its own; its pieces of
// kSlChunk entries are summed by the gather's blocks straight from x.
// Per entry the streams are 2 bytes of column, 2 of position, and the value
// written and read back.  The gather is bound by them; the rows kernel waits
// on the chain run start -> value -> LDS -> sum of each chunk.
// Configuration model, n = 10^7, 75.7 M entries, unit weights: FP32 0.35 ms
// per apply (gather 0.12, 4.9 TB/s; rows 0.23, 2.7 TB/s) against 0.69 for the
// L2 slices and 1.26 row by row; FP64 0.59 ms (0.22 and 0.37) against 1.09
// and 1.37.
// Every sum is taken in a fixed order, so results repeat bit for bit.  The
// order of the entries is built on the host from the graph's CSR the first
// time it is needed and kept with the graph; it does not depend on the
// weights.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <string>
#include <thread>
#include <vector>

#include "device_common.hpp"
#include "prof.hpp"

namespace nvd {

constexpr int kSlBS = 1024;
// Nodes per slice: two FP32 slices (two blocks) or one FP64 slice fill a CU's
// 160 KB of LDS.
constexpr int kSlNodes = 20352;
// CSR entries per chunk (the LDS values of the rows kernel: two FP32 blocks or
// one FP64 block per CU, beside the reductions' scratch).
constexpr int kSlChunk = 16384;
// Entries above which a row is summed by a group of 16 lanes, and by its wave.
constexpr int kSlGroupRow = 16;
constexpr int kSlWaveRow = 256;
// Graphs this large try the slices by default.  Below, x stays near enough (us row
// by row / sliced: power law n = 5.2 10^5 FP64 45 / 47, FP32 35 / 40, n = 2.6 10^5
// 25 / 58 and 22 / 53; ER n = 5.2 10^5 of degree 6 23 / 43); from here on it
// depends on the graph, and both are timed (power law n = 1.05 10^6 93 / 63 and 66
// / 43; BA n = 1.3 10^6 87 / 152 and 59 / 89).
constexpr int kSlMinN = 1 << 20;
// Blocks of both kernels: what 256 CUs hold at once.
template <typename V>
constexpr int kSlBlocks = sizeof(V) == 8 ? 256 : 512;

struct SliceGraph {
  int S = 0, nch = 0, sn = 0, lsh = 0;
  unsigned quads = 0;              // entries / 4 (every slice padded to a multiple of 4)
  unsigned* off4 = nullptr;        // [S+1] first entry of slice s, / 4
  uint16_t* lcol = nullptr;        // [4 quads] column within the slice
  uint16_t* pos = nullptr;         // [4 quads] CSR position within the chunk
  unsigned* run = nullptr;         // [nch+1][S] first entry of chunk c in slice s
  int* row0 = nullptr;             // [nch+1] first row of chunk c
  int* piece0 = nullptr;           // [nch+1] first piece of a chunk that is one long row
  int n_piece = 0;
  int* piece = nullptr;            // [n_piece][3] row, CSR range
  double* val = nullptr;           // [4 quads] neighbours' values, FP32 or FP64
  double* psum = nullptr;          // [n_piece]
  int64_t bytes = 0;
};

struct SliceArgs {
  int n, S, nch, sn, lsh, n_piece;
  unsigned quads;
  const unsigned* off4;
  const uint16_t* lcol;
  const uint16_t* pos;
  const unsigned* run;
  const int* row0;
  const int* piece0;
  const int* piece;
  void* val;
  double* psum;
  const int* rp;
  const int* ci;
  const void* w;     // CSR weights in the call's precision
  const int* gate;   // EPI_CG: the tile's active count; nothing to do when 0
};

template <typename V>
struct SliceOut {
  const V* x;
  long ldx;
  V* y;
  long ldy;
  const double* b;
  long ldb;
  ColState* cs;
};

__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum over the 16 lanes of a DPP row, in every lane of it.
template <int CTRL>
__device__ __forceinline__ double row_turned(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double group_total(double v) {
  v += row_turned<0x128>(v);   // row_ror:8, 4, 2, 1
  v += row_turned<0x124>(v);
  v += row_turned<0x122>(v);
  v += row_turned<0x121>(v);
  return v;
}

template <typename V, bool UNIT>
__global__ __launch_bounds__(kSlBS, sizeof(V) == 8 ? 4 : 8) void k_slice_gather(SliceArgs a, const V* __restrict__ x,
                                                                               long ldx) {
  extern __shared__ double lds[];
  V* xs = reinterpret_cast<V*>(lds);
  if (a.gate && *a.gate == 0) return;
  const int t = threadIdx.x;
  const unsigned per = (a.quads + gridDim.x - 1) / gridDim.x;
  unsigned q = min(a.quads, blockIdx.x * per);
  const unsigned qend = min(a.quads, q + per);
  int s = 0;
  for (int lo = 0, hi = a.S; lo < hi;) {   // last slice that starts at or before q
    const int mid = (lo + hi) >> 1;
    if (a.off4[mid + 1] <= q) {
      lo = mid + 1;
    } else {
      hi = mid;
    }
    s = lo;
  }
  const uint2* lc = reinterpret_cast<const uint2*>(a.lcol);
  using V4 = typename VecOf<V, 4>::type;
  V4* out = static_cast<V4*>(a.val);
  for (; q < qend; ++s) {
    const unsigned qs = min(qend, a.off4[s + 1]);
    if (qs == q) continue;
    const long j0 = (long)s * a.sn;
    const int m = (int)min((long)a.sn, a.n - j0);
#pragma unroll 4
    for (int j = t; j < m; j += kSlBS) xs[j] = x[(j0 + j) * ldx];
    __syncthreads();
    unsigned i = q + t;
    constexpr int U = 4;
    for (; i + (U - 1) * kSlBS < qs; i += U * kSlBS) {
      uint2 c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = lc[i + u * kSlBS];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        V4 v;
        v[0] = xs[c[u].x & 0xffffu];
        v[1] = xs[c[u].x >> 16];
        v[2] = xs[c[u].y & 0xffffu];
        v[3] = xs[c[u].y >> 16];
        out[i + u * kSlBS] = v;
      }
    }
    for (; i < qs; i += kSlBS) {
      const uint2 c = lc[i];
      V4 v;
      v[0] = xs[c.x & 0xffffu];
      v[1] = xs[c.x >> 16];
      v[2] = xs[c.y & 0xffffu];
      v[3] = xs[c.y >> 16];
      out[i] = v;
    }
    __syncthreads();
    q = qs;
  }
  // pieces of long rows
  const V* w = static_cast<const V*>(a.w);
  for (int p = blockIdx.x; p < a.n_piece; p += gridDim.x) {
    const int row = a.piece[3 * p], lo = a.piece[3 * p + 1], hi = a.piece[3 * p + 2];
    const double xv = (double)x[row * ldx];
    double sum = 0.0;
#pragma unroll 4
    for (int e = lo + t; e < hi; e += kSlBS)
      sum += (UNIT ? 1.0 : (double)w[e]) * (xv - (double)x[a.ci[e] * ldx]);
    sum = wave_total(sum);
    if ((t & 63) == 0) lds[t >> 6] = sum;
    __syncthreads();
    if (t == 0) {
      double tot = 0.0;
      for (int k = 0; k < kSlBS / 64; ++k) tot += lds[k];
      a.psum[p] = tot;
    }
    __syncthreads();
  }
}

template <typename V, bool UNIT, int EPI>
__global__ __launch_bounds__(kSlBS, sizeof(V) == 8 ? 4 : 8) void k_slice_rows(SliceArgs a, SliceOut<V> o, GridRed red) {
  constexpr int ND = EPI == EPI_CG ? 1 : (EPI == EPI_RESID ? 5 : 0);
  constexpr int NDA = ND > 0 ? ND : 1;
  extern __shared__ double lds[];
  __shared__ double vals[NDA];
  V* xe = reinterpret_cast<V*>(lds);
  if constexpr (EPI == EPI_CG) {
    if (o.cs->n_active == 0) return;
  }
  const int t = threadIdx.x, lane = t & 63;
  const V* w = static_cast<const V*>(a.w);
  const V* val = static_cast<const V*>(a.val);
  double dacc[NDA][1];
#pragma unroll
  for (int d = 0; d < NDA; ++d) dacc[d][0] = 0.0;
  auto finish = [&](unsigned row, double xv, double sum) {
    const V yv = (V)sum;
    if constexpr (EPI == EPI_PLAIN) {
      o.y[row * o.ldy] = yv;
    } else if constexpr (EPI == EPI_CG) {
      o.y[row * o.ldy] = yv;
      dacc[0][0] += xv * (double)yv;
    } else {
      const double bb = o.b[row * o.ldb];
      const double rr = bb - (double)yv;
      o.y[row * o.ldy] = (V)rr;
      dacc[0][0] += bb * xv;
      dacc[1][0] += xv * rr;
      dacc[2][0] += rr * rr;
      dacc[3][0] += rr;
      dacc[4][0] += xv;
    }
  };
  // block b runs on XCD b mod 8 (the grid is a multiple of 8): the chunks of
  // an XCD are consecutive, and its blocks walk them side by side
  const int xcd = blockIdx.x & 7;
  const int c1 = (int)((long)(xcd + 1) * a.nch / 8);
  const int nsub = kSlBS >> a.lsh, sub = t >> a.lsh, l = t & ((1 << a.lsh) - 1);
  for (int c = (int)((long)xcd * a.nch / 8) + (blockIdx.x >> 3); c < c1; c += gridDim.x >> 3) {
    const unsigned r0 = a.row0[c], r1 = a.row0[c + 1];
    const int pc = a.piece0[c], pn = a.piece0[c + 1];
    if (pn > pc) {   // one long row
      if (t < 64) {
        double sum = 0.0;
        for (int p = pc + lane; p < pn; p += 64) sum += a.psum[p];
        sum = wave_total(sum);
        if (t == 0) finish(r0, (double)o.x[r0 * o.ldx], sum);
      }
      continue;
    }
    // the thread's first row, in flight while the values arrive
    unsigned row = (unsigned)r0 + t;
    int e0 = 0, e1 = 0;
    V xv = (V)0;
    if (row < r1) {
      e0 = a.rp[row];
      e1 = a.rp[row + 1];
      xv = o.x[row * o.ldx];
    }
    const int ebase = a.rp[r0];
    const unsigned* run = a.run + (long)c * a.S;
    constexpr int U = 4;   // runs in flight; 8 spill in FP32: 415 us per apply against 350
    for (int s = sub; s < a.S; s += U * nsub) {
      unsigned p[U], e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int su = s + u * nsub;
        const bool in = su < a.S;
        p[u] = in ? run[su] + l : 0u;
        e[u] = in ? run[su + a.S] : 0u;
      }
      bool more = true;
      while (more) {
        V v[U];
        unsigned at[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p[u] < e[u]) {
            v[u] = val[p[u]];
            at[u] = a.pos[p[u]];
          }
        more = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (p[u] < e[u]) xe[at[u]] = v[u];
          p[u] += 1u << a.lsh;
          more = more || p[u] < e[u];
        }
      }
    }
    __syncthreads();
    const int rows = (int)(r1 - r0);
    for (int base = 0; base < rows; base += kSlBS) {
      const unsigned next = row + kSlBS;
      int f0 = 0, f1 = 0;
      V xn = (V)0;
      if (next < r1) {
        f0 = a.rp[next];
        f1 = a.rp[next + 1];
        xn = o.x[next * o.ldx];
      }
      const double xr = (double)xv;
      const int len = e1 - e0;
      double sum = 0.0;
      if (len <= kSlGroupRow) {
        for (int j = 0; j < len; j += 4) {
          double term[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = min(e0 + j + u, e1 - 1);
            term[u] = (UNIT ? 1.0 : (double)w[e]) * (xr - (double)xe[e - ebase]);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) sum += j + u < len ? term[u] : 0.0;
        }
      }
      // four rows at a time, 16 lanes each: group i takes the i-th of the mask
      for (unsigned long long m = __ballot(len > kSlGroupRow && len <= kSlWaveRow); m != 0;) {
        const int mine = __popcll(m & ((1ull << lane) - 1ull));
        const bool out = (m >> lane & 1ull) != 0 && mine < 4;
        const unsigned long long m1 = m & (m - 1), m2 = m1 & (m1 - 1), m3 = m2 & (m2 - 1);
        const int grp = lane >> 4;
        const unsigned long long mg = grp == 0 ? m : (grp == 1 ? m1 : (grp == 2 ? m2 : m3));
        const int k = mg != 0 ? __builtin_ctzll(mg) : lane;
        const int b0 = __shfl(e0, k, 64), b1 = __shfl(e1, k, 64);   // (in every lane: its source must be active)
        const double xb = __shfl(xr, k, 64);
        double part = 0.0;
        for (int e = b0 + (lane & 15); e < (mg != 0 ? b1 : b0); e += 16)
          part += (UNIT ? 1.0 : (double)w[e]) * (xb - (double)xe[e - ebase]);
        part = __shfl(group_total(part), mine << 4 & 63, 64);
        if (out) sum = part;
        m = m3 & (m3 - 1);
      }
      for (unsigned long long m = __ballot(len > kSlWaveRow); m != 0; m &= m - 1) {
        const int k = __builtin_ctzll(m);
        const int b0 = __shfl(e0, k, 64), b1 = __shfl(e1, k, 64);
        const double xb = __shfl(xr, k, 64);
        double part = 0.0;
        for (int e = b0 + lane; e < b1; e += 64)
          part += (UNIT ? 1.0 : (double)w[e]) * (xb - (double)xe[e - ebase]);
        part = wave_total(part);
        if (lane == k) sum = part;
      }
      if (row < r1) finish(row, xr, sum);
      row = next;
      e0 = f0;
      e1 = f1;
      xv = xn;
    }
    __syncthreads();
  }
  if constexpr (ND > 0) {
    __syncthreads();
    block_reduce_cols<kSlBS, ND, 1>(dacc, 1, lds);
    if (t == 0) {
#pragma unroll
      for (int d = 0; d < ND; ++d) vals[d] = lds[d * kSlBS];
    }
    __syncthreads();
    if (!grid_reduce<kSlBS>(vals, ND, red)) return;
    if (t == 0) {
      ColState* cs = o.cs;
      if constexpr (EPI == EPI_CG) {
        const double sg = vals[0];
        double al = 0.0;
        if (cs->active[0]) {
          if (!(sg > 0.0) || !isfinite(sg)) {
            cs->status[0] = kStBreak;
            cs->active[0] = 0;
            cs->oactive[0] = 0;
          } else {
            al = cs->rho[0] / sg;
          }
        }
        cs->alpha[0] = al;
      } else {
#pragma unroll
        for (int d = 0; d < ND; ++d) cs->dots[d][0] = vals[d];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host: build, use, free
// ---------------------------------------------------------------------------
void free_slices(DevGraph* g) {
  SliceGraph* sg = g->slices;
  if (!sg) return;
  (void)hipDeviceSynchronize();
  void* ps[] = {sg->off4, sg->lcol, sg->pos, sg->run, sg->row0, sg->piece0, sg->piece, sg->val, sg->psum};
  for (void* p : ps)
    if (p) (void)hipFree(p);
  g->bytes -= sg->bytes;
  delete sg;
  g->slices = nullptr;
  g->slice_state = 0;
}

// NVD_SLICE: "0" never, "1" for every graph, otherwise graphs of at least
// kSlMinN nodes.  NVD_SLICE_NODES: nodes per slice (default and most kSlNodes).
static int slice_mode() {
  const char* e = std::getenv("NVD_SLICE");
  if (e && e[0] == '0') return 0;
  if (e && e[0] == '1') return 1;
  return 2;
}

bool slices_serve(const DevGraph* g) {
  const int mode = slice_mode();
  return mode == 1 || (mode == 2 && g->n >= kSlMinN);
}

template <typename T>
static bool room(T** dst, size_t count, int64_t& bytes) {
  const size_t nb = std::max<size_t>(1, count) * sizeof(T);
  if (hipMalloc(reinterpret_cast<void**>(dst), nb) != hipSuccess) {
    *dst = nullptr;
    return false;
  }
  bytes += (int64_t)nb;
  return true;
}

template <typename T>
static bool up(T** dst, const std::vector<T>& v, int64_t& bytes) {
  return room(dst, v.size(), bytes) &&
         (v.empty() || hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice) == hipSuccess);
}

static nvd_status build_slices(DevGraph* g) {
  const long n = g->n;
  long sn = kSlNodes;
  if (const char* e = std::getenv("NVD_SLICE_NODES")) {
    const long v = std::atol(e);
    if (v >= 1 && v < sn) sn = v;
  }
  const std::vector<int>& rp = g->h_rp;
  const std::vector<int>& ci = g->h_ci;
  const int S = (int)((n + sn - 1) / sn);
  // chunks: as many rows as kSlChunk entries hold, and no more than kSlChunk
  // rows (isolated nodes have no entries); a longer row by itself
  std::vector<int> row0(1, 0), piece0(1, 0), piece;
  for (long r = 0; r < n;) {
    long e = r + 1;
    if (rp[e] - rp[r] > kSlChunk) {
      for (long lo = rp[r]; lo < rp[e]; lo += kSlChunk) {
        piece.push_back((int)r);
        piece.push_back((int)lo);
        piece.push_back((int)std::min<long>(lo + kSlChunk, rp[e]));
      }
    } else {
      while (e < n && rp[e + 1] - rp[r] <= kSlChunk && e - r < kSlChunk) ++e;
    }
    row0.push_back((int)e);
    piece0.push_back((int)(piece.size() / 3));
    r = e;
  }
  const int nch = (int)row0.size() - 1;
  // Runs of three to four entries (10^8 nodes, 7.6 10^8 entries) no longer pay: n =
  // 1.3 10^8, ms sliced / row by row, FP32 23.2 / 19.9, FP64 17.9 / 19.0.
  if ((long)S * (nch + 1) > (1L << 28)) {
    set_error("slices: graph too large for the sliced apply");
    return NVD_E_UNSUPPORTED;
  }
  const int nthr = (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
  auto chunks = [&](auto&& f) {
    std::vector<std::thread> th;
    for (int tt = 0; tt < nthr; ++tt)
      th.emplace_back([&, tt] {
        for (int c = tt; c < nch; c += nthr)
          if (piece0[c + 1] == piece0[c]) f(c);
      });
    for (auto& x : th) x.join();
  };
  // entries of each (chunk, slice), then where each run starts
  std::vector<unsigned> run((size_t)S * (nch + 1), 0u);
  chunks([&](int c) {
    unsigned* cnt = &run[(size_t)S * c];
    for (long e = rp[row0[c]]; e < rp[row0[c + 1]]; ++e) cnt[ci[e] / sn]++;
  });
  std::vector<unsigned> at(S, 0u), off4(S + 1, 0u);
  for (int c = 0; c < nch; ++c)
    for (int s = 0; s < S; ++s) at[s] += run[(size_t)S * c + s];
  unsigned total = 0;
  for (int s = 0; s < S; ++s) {
    const unsigned len = at[s];
    at[s] = total;
    off4[s] = total / 4;
    total += (len + 3) / 4 * 4;
  }
  off4[S] = total / 4;
  for (int c = 0; c <= nch; ++c)
    for (int s = 0; s < S; ++s) {
      const unsigned len = run[(size_t)S * c + s];
      run[(size_t)S * c + s] = at[s];
      at[s] += len;
    }
  std::vector<uint16_t> lcol(total, 0), pos(total, 0);
  chunks([&](int c) {
    std::vector<unsigned> next(run.begin() + (size_t)S * c, run.begin() + (size_t)S * (c + 1));
    const long e0 = rp[row0[c]];
    for (long e = e0; e < rp[row0[c + 1]]; ++e) {
      const int s = (int)(ci[e] / sn);
      const unsigned p = next[s]++;
      lcol[p] = (uint16_t)(ci[e] - s * sn);
      pos[p] = (uint16_t)(e - e0);
    }
  });
  SliceGraph* sg = new SliceGraph();
  sg->S = S;
  sg->nch = nch;
  sg->sn = (int)sn;
  sg->quads = total / 4;
  sg->n_piece = (int)(piece.size() / 3);
  // lanes per run: at most half its average, so that few of the last step's
  // lanes are idle, and at most 16 (10^7 nodes, runs of 33: FP32 apply 350 us
  // with 16 lanes, 394 with 8, whose loads are half as wide)
  const double avg = (double)total / ((double)S * nch);
  while (sg->lsh < 4 && (4 << sg->lsh) <= avg) sg->lsh++;
  const bool ok = up(&sg->off4, off4, sg->bytes) && up(&sg->lcol, lcol, sg->bytes) && up(&sg->pos, pos, sg->bytes) &&
                  up(&sg->run, run, sg->bytes) && up(&sg->row0, row0, sg->bytes) &&
                  up(&sg->piece0, piece0, sg->bytes) && up(&sg->piece, piece, sg->bytes) &&
                  room(&sg->val, total, sg->bytes) && room(&sg->psum, (size_t)sg->n_piece, sg->bytes);
  g->slices = sg;
  g->bytes += sg->bytes;
  if (!ok) {
    (void)hipGetLastError();
    free_slices(g);
    set_error("slices: device allocation failed");
    return NVD_E_NOMEM;
  }
  return NVD_OK;
}

template <typename V, bool UNIT, int EPI>
static nvd_status launch_forms(const SliceArgs& a, const SliceOut<V>& o, const GridRed& red, hipStream_t s) {
  constexpr int lds_gather = kSlNodes * sizeof(V), lds_rows = kSlChunk * sizeof(V);
  auto* gather = &k_slice_gather<V, UNIT>;
  auto* rows = &k_slice_rows<V, UNIT, EPI>;
  NVD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(gather), hipFuncAttributeMaxDynamicSharedMemorySize,
                              lds_gather));
  NVD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(rows), hipFuncAttributeMaxDynamicSharedMemorySize,
                              lds_rows));
  gather<<<kSlBlocks<V>, kSlBS, lds_gather, s>>>(a, o.x, o.ldx);
  rows<<<std::min(kSlBlocks<V>, (a.nch + 7) / 8 * 8), kSlBS, lds_rows, s>>>(a, o, red);
  NVD_HIP(hipGetLastError());
  return NVD_OK;
}

template <typename V, bool UNIT>
static nvd_status launch_epi(const SliceArgs& a, const SliceOut<V>& o, int epi, const GridRed& red, hipStream_t s) {
  switch (epi) {
    case EPI_PLAIN: return launch_forms<V, UNIT, EPI_PLAIN>(a, o, red, s);
    case EPI_CG: return launch_forms<V, UNIT, EPI_CG>(a, o, red, s);
    case EPI_RESID:
      if constexpr (sizeof(V) == 8) return launch_forms<V, UNIT, EPI_RESID>(a, o, red, s);
      break;
    default: break;
  }
  set_error("slices: unsupported epilogue");
  return NVD_E_UNSUPPORTED;
}

template <typename V>
static nvd_status launch_sliced(const SpmmCall& c, const GridRed& red, hipStream_t s) {
  const DevGraph* g = c.g;
  const SliceGraph* sg = g->slices;
  const bool unit = !g->weighted;
  SliceArgs a{};
  a.n = g->n;
  a.S = sg->S;
  a.nch = sg->nch;
  a.sn = sg->sn;
  a.lsh = sg->lsh;
  a.n_piece = sg->n_piece;
  a.quads = sg->quads;
  a.off4 = sg->off4;
  a.lcol = sg->lcol;
  a.pos = sg->pos;
  a.run = sg->run;
  a.row0 = sg->row0;
  a.piece0 = sg->piece0;
  a.piece = sg->piece;
  a.val = sg->val;
  a.psum = sg->psum;
  a.rp = g->rp;
  a.ci = g->ci;
  if constexpr (sizeof(V) == 8)
    a.w = g->w64;
  else
    a.w = g->w32;
  a.gate = c.epi == EPI_CG ? &c.cs->n_active : nullptr;
  SliceOut<V> o{};
  o.x = static_cast<const V*>(c.x);
  o.ldx = c.ldx;
  o.y = static_cast<V*>(c.y);
  o.ldy = c.ldy;
  o.b = c.b;
  o.ldb = c.ldb;
  o.cs = c.cs;
  int pid = -1;
  if (prof_enabled()) {
    const double sv = (double)sizeof(V);
    const double sw = unit ? 0.0 : sv;
    const double n = g->n;
    const double csr = (4.0 + sw) * g->nnz + 4.0 * (n + 1);
    const double vecb = c.epi == EPI_RESID ? 3.0 * 8.0 * n : 2.0 * sv * n;
    pid = prof_begin(s, sizeof(V) == 8 ? PK_SPMM64 : PK_SPMM32, csr + vecb);
  }
  const nvd_status st = unit ? launch_epi<V, true>(a, o, c.epi, red, s) : launch_epi<V, false>(a, o, c.epi, red, s);
  prof_end(s, pid);
  return st;
}

// For nvd_laplacian_apply the sliced form has to be faster by a tenth: on one x
// again and again, both run from warm caches, which the row-wise one is the less
// dependent on (ER n = 1.065 10^6 of degree 3, weighted, FP64, us row by row /
// sliced: timed so 42.7 / 41.0, with a new x each time 43.0 / 45.7).  A solve's x
// was written by the kernel before, and there the faster one is taken (whole calls
// on that graph 16.1 / 14.9 ms; power law n = 1.16 10^6, weighted, FP64, timed 138 /
// 137 us, in its solve 138 / 131 and the call 6.53 / 6.28 ms).
constexpr float kSlGain = 0.9f;

// Time the row-wise and the sliced apply of this call's x (EPI_PLAIN into a
// scratch y, 3 launches each after a warm-up).
template <typename V>
static nvd_status time_forms(DevGraph* g, const SpmmCall& c, const GridRed& red, hipStream_t s, float* t_row,
                             float* t_sliced) {
  void* y = nullptr;
  NVD_HIP(hipMalloc(&y, sizeof(V) * (size_t)g->n));
  SpmmCall t = c;
  t.epi = EPI_PLAIN;
  t.y = y;
  t.ldy = 1;
  t.b = nullptr;
  t.cs = nullptr;
  hipEvent_t a = nullptr, b = nullptr;
  nvd_status st = hipEventCreate(&a) == hipSuccess && hipEventCreate(&b) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
  for (int form = 0; form < 2 && st == NVD_OK; ++form) {
    auto run = [&]() { return form == 0 ? launch_spmm(t, red, s) : launch_sliced<V>(t, red, s); };
    st = run();
    if (st == NVD_OK) st = hipEventRecord(a, s) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
    for (int i = 0; i < 3 && st == NVD_OK; ++i) st = run();
    if (st == NVD_OK) st = hipEventRecord(b, s) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
    if (st == NVD_OK) st = hipEventSynchronize(b) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
    float ms = 0.0f;
    if (st == NVD_OK) st = hipEventElapsedTime(&ms, a, b) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
    (form == 0 ? *t_row : *t_sliced) = ms;
  }
  if (a) (void)hipEventDestroy(a);
  if (b) (void)hipEventDestroy(b);
  (void)hipStreamSynchronize(s);
  (void)hipFree(y);
  return st;
}

// The sliced apply serves T = 1 on graphs of at least kSlMinN nodes where it
// is the faster form: the first eligible call of each precision builds the
// slices (state -1 after a failed build: the graph keeps the row-wise apply)
// and times both forms.  Calls with a bounded SpMM grid keep the row-wise
// apply.
static bool use_slices(DevGraph* g, const SpmmCall& c, const GridRed& red, hipStream_t s) {
  // a caller that bounds the grid (the no-allocation entry point) has sized
  // its reduction scratch for it, and building the slices would allocate
  if (c.T != 1 || g->n < 1 || c.grid > 0) return false;
  if (!slices_serve(g) || g->slice_state < 0) return false;
  const int mode = slice_mode();
  const int p = c.prec == 0 ? 0 : 1;
  if (mode == 2 && g->slice_pick[p] < 0) return false;
  if (!g->slices) {
    if (build_slices(g) != NVD_OK) {
      g->slice_state = -1;
      return false;
    }
    g->slice_state = 1;
  }
  if (mode == 2 && g->slice_pick[p] == 0) {
    float tr = 0.0f, ts = 0.0f;
    const nvd_status st = c.prec == 0 ? time_forms<double>(g, c, red, s, &tr, &ts)
                                      : time_forms<float>(g, c, red, s, &tr, &ts);
    g->slice_pick[p] = st != NVD_OK || ts >= tr ? -1 : (ts < kSlGain * tr ? 2 : 1);
    if (g->slice_pick[0] < 0 && g->slice_pick[1] < 0) {
      free_slices(g);
      return false;
    }
  }
  return mode == 1 || g->slice_pick[p] > (c.epi == EPI_PLAIN ? 1 : 0);
}

nvd_status launch_apply(const SpmmCall& c, const GridRed& red, hipStream_t s) {
  if (c.g->n == 0) return NVD_OK;
  DevGraph* g = const_cast<DevGraph*>(c.g);
  if (use_slices(g, c, red, s)) return c.prec == 0 ? launch_sliced<double>(c, red, s) : launch_sliced<float>(c, red, s);
  return launch_spmm(c, red, s);
}

}  // namespace nvd
