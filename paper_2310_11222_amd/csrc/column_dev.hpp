// Device side of the one-block-per-column solver (column.hip): the graph's
// layout as a block reads it, block-wide sums, the Laplacian rows and the CG
// loop.
#pragma once

#include <type_traits>

#include "device_common.hpp"
#include "refine_guard.hpp"

namespace nvd {

constexpr int kColBS = 1024;
constexpr int kColWaves = kColBS / 64;

// A graph as one block walks it.  Positions are the nodes in order of falling
// degree (perm: position -> node).  Positions 64 s .. 64 s + 63 form slice s,
// whose rows are stored as pairs of neighbour positions, one pair of every
// row side by side (a "pair row" of 64: a wave reads 256 contiguous bytes),
// as many as its longest row needs; a missing neighbour is the row's own
// position, which adds w (p_i - p_i) = 0.  Wave w takes slices w, w + 16, ...
// (slot j: slice w + 16 j), whose pair rows follow each other in memory.
//
// The first nh positions are heavy rows, whose neighbours are cut into parts
// of equal length, each a row of its own (nv parts, in vslots further slots)
// whose sum goes to LDS, where the heavy row's owner adds its parts.  A hub
// then costs the block what its entries cost and not the length of its row
// (a wave for each heavy row took 1.5 of 3.3 us an iteration on a 10^3-node
// preferential-attachment graph).
struct ColGraph {
  int n, nh, nv, nc;
  int slots, vslots;             // slices of a wave: positions, parts of heavy rows
  int nc_block, nc_wave;         // components (largest first) summed by the block, by a wave
  const int* perm;               // [n]
  const int* soff;               // [16 (slots + vslots) + 1] first pair row of (wave, slot)
  const unsigned* idx;           // [pair rows][64]
  const double2* w64;            // [pair rows][64] (null: unit weights)
  const float2* w32;
  const int* voff;               // [nh + 1] parts of each heavy row
  const int* vown;               // [1024 vslots] heavy row of each part
  const double* inv64;           // [slots * 1024] 1 / degree by position (0: isolated, past n)
  const float* inv32;
  const int* coff;               // [nc + 1] members of each component (nc > 1)
  const int* cnode;              // [n] positions, grouped by component
  const int* ccomp;              // [n] component of each position
};

constexpr int kColSpare = 3;     // pair rows a stream reads past its end

template <typename T>
__device__ __forceinline__ void make_scalar(T*& p) {
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  p = reinterpret_cast<T*>(((unsigned long long)hi << 32) | lo);
}

// A block's graph, in scalar registers whichever table it came from.
__device__ __forceinline__ void make_scalar(ColGraph& g) {
  for (int* v : {&g.n, &g.nh, &g.nv, &g.nc, &g.slots, &g.vslots, &g.nc_block, &g.nc_wave})
    *v = __builtin_amdgcn_readfirstlane(*v);
  make_scalar(g.perm);
  make_scalar(g.soff);
  make_scalar(g.idx);
  make_scalar(g.w64);
  make_scalar(g.w32);
  make_scalar(g.voff);
  make_scalar(g.vown);
  make_scalar(g.inv64);
  make_scalar(g.inv32);
  make_scalar(g.coff);
  make_scalar(g.cnode);
  make_scalar(g.ccomp);
}

constexpr int kColNoEvent = 0x7fff;
enum { kColPreTree = 1, kColPreAchol = 2 };

// An explicit preconditioner in the block's order (column_pre.hip).
struct ColPre {
  int kind;
  // approximate Cholesky: forward (0) and backward (1) solve
  const unsigned short* apos;    // [n] elimination position of each position
  const int4* steps[2];          // nsteps + 2 (empty ones last)
  int nsteps[2];
  const unsigned short* idx[2];
  const double* c64[2];
  const float* c32[2];
  const double* ip64;            // [n] 1 / pivot by elimination position
  const float* ip32;
  // spanning forest, by position: preorder place, subtree size, the
  // component's first and last preorder place, 1 / weight to the parent
  const unsigned short *tpre, *tsize, *tlo, *thi;
  const double* twinv;
  const unsigned short* tour;    // [2 slots][1024] events: preorder place, 0x8000: left
  int k, nend;                   // augmenting edges, nodes they touch
  const unsigned short* auv;     // [2k] preorder places of their ends
  const double* Cinv;            // [k][k]
  const int* aoff;               // [nend + 1]
  const unsigned short* aend;    // [nend] preorder place
  const unsigned short* aedge;   // edge, 0x8000: its second end
};

// One column to solve: pair data at P[voff + i * ld], results at `out`.
struct ColJob {
  int graph;
  int out;
  long voff;
  long ld;
  long xoff;     // X[xoff + i * ldx]
  long ldx;
  long work;     // its vectors in vec
};

// Whose pairs a launch solves.  A graph's own call: a pair whose CG run ends at
// max_iter has not converged, one that FP32 cannot finish is left to an FP64
// launch, and FP64 takes up to three runs.  A batch's: a run that ends at max_iter
// counts, and the next goes on from its x; FP64 takes up to three, or two (mixed
// precision: kColBatch).  One value, and a constant bound on the runs, as every
// scalar more that the kernel holds costs its FP64 form registers (n = 10^4 of
// degree 16, weighted, 5 pairs: 1122 us with the runs and the rest apart, 1106).
enum ColCall : int { kColBatch = 0, kColOwn, kColBatchTwo };

struct ColArgs {
  ColGraph g;                // the graph, unless `graphs` is set
  ColPre pre;                // its preconditioner (one graph only)
  int vecs;                  // vectors of a block in vec: 4, with a preconditioner 8
  const ColGraph* graphs;    // several graphs: jobs[block] names the one
  const ColJob* jobs;        // null: block b takes column col0 + b of g
  const double* P;
  const double* Q;           // null: P alone
  long ld;
  int col0;
  double rtol2, irtol2, stall_ratio2;
  int max_iter, out_dsq, max_refine;
  int lds_n;                 // FP64 values that fit the gathered vector's LDS
  int call;                  // ColCall
  int resume;                // FP64: only those pairs, from their x in vec
  double* d_out;
  double* X;                 // null, or n x k (ldx) for the solutions; the same
  double* B;                 // for delta_bar
  double* R;                 // and for the final residuals
  long ldx;
  nvd_pair_info* info;       // pinned host memory, one per block from info0
  double* vec;               // [blocks][vecs][stride] b, x, r, FP32 x, scratch
  long stride;
  double* cmean;             // [blocks][cstride] component means (nc > 1)
  long cstride;
};

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Sum over each row of 16 lanes, the same in all of them: register moves
// between lanes (swap pairs, swap pairs of pairs, mirror 8, mirror 16)
// instead of the 40-cycle LDS round trip of a shuffle.
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  return v;
}

// Sum over the wave in a fixed order, the same in every lane.
__device__ __forceinline__ double wave_total(double v) {
  v = row16_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

struct ColShared {
  double part[2][5][kColWaves];
};

// Block sums of ND values, the same in every thread.  Two sets of partials
// take turns, so one barrier is enough: a set is written again only after
// the barrier of the reduction between, which every reader has passed.
template <int ND>
__device__ __forceinline__ void col_sum(double (&v)[ND], ColShared& S, int& turn) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < ND; ++d) v[d] = wave_total(v[d]);
  if (lane == 0) {
#pragma unroll
    for (int d = 0; d < ND; ++d) S.part[turn][d][w] = v[d];
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < ND; ++d) v[d] = row16_sum(S.part[turn][d][lane & 15]);
  turn ^= 1;
}

__device__ __forceinline__ bool uniform(bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; }

template <typename V>
struct ColW;
template <>
struct ColW<double> {
  using V2 = double2;
  static __device__ const double2* slices(const ColGraph& g) { return g.w64; }
  static __device__ const double* inv(const ColGraph& g) { return g.inv64; }
};
template <>
struct ColW<float> {
  using V2 = float2;
  static __device__ const float2* slices(const ColGraph& g) { return g.w32; }
  static __device__ const float* inv(const ColGraph& g) { return g.inv32; }
};

// Between the unrolled elements of a thread: keeps the compiler from loading
// ahead for all of them at once, which spills the vectors held in registers.
template <int EPT>
__device__ __forceinline__ void four_at_a_time(int j) {
  if (EPT > 4 && (j & 3) == 3) asm volatile("" ::: "memory");
}

// The thread's index (the wave's, in a scalar register), opaque to the
// compiler at this place: addresses formed from it are formed where they are
// used, not kept in registers for every element across the iterations.
__device__ __forceinline__ int thread_here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ int wave_here() {
  int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  asm volatile("" : "+s"(w));
  return w;
}

// The wave's pair rows as one stream over its slots, read D rows ahead: while
// a pair is gathered, the indices and weights of the next ones (of the same
// slice or of the next) are on their way from L2.  The loads are
// unconditional (the stream ends in D spare rows), so a step is straight
// code; steps of several rows with a test for each were slower.
template <typename V, bool UNIT>
struct ColStream {
  using V2 = typename ColW<V>::V2;
  static constexpr int D = sizeof(V) == 8 && !UNIT ? 2 : 3;
  const unsigned* ix;
  const V2* wx;
  unsigned a[D];
  V2 w[UNIT ? 1 : D];

  static __device__ __forceinline__ int lane_int(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

  __device__ __forceinline__ void start(const ColGraph& g, int first) {
    const size_t at = (size_t)lane_int(first, 0) * 64;
    const unsigned l = threadIdx.x & 63;
    ix = g.idx + at;
    wx = UNIT ? nullptr : ColW<V>::slices(g) + at;
#pragma unroll
    for (int u = 0; u < D; ++u) {
      a[u] = ix[u * 64 + l];
      if constexpr (!UNIT) w[u] = wx[u * 64 + l];
    }
  }
  // The lane's row of L in slot j, in edge differences: sum_j w_ij (p_i - p_j)
  // with p in LDS or in memory; `first` holds the slots' offsets by lane.
  // PART: only the neighbours in positions [base, base + count), p holding
  // those.
  template <bool PART = false>
  __device__ __forceinline__ V row(int first, int j, const V* p, V pi, unsigned base = 0, unsigned count = 0) {
    const unsigned l = threadIdx.x & 63;
    V sum = (V)0;
#pragma unroll 1
    for (int left = lane_int(first, j + 1) - lane_int(first, j); left > 0; --left) {
      V v0, v1;
      if constexpr (PART) {
        const unsigned i0 = (a[0] & 0xffffu) - base, i1 = (a[0] >> 16) - base;
        v0 = i0 < count ? p[i0] : pi;
        v1 = i1 < count ? p[i1] : pi;
      } else {
        v0 = p[a[0] & 0xffffu];
        v1 = p[a[0] >> 16];
      }
      V2 w0;
      if constexpr (!UNIT) w0 = w[0];
#pragma unroll
      for (int u = 0; u + 1 < D; ++u) {
        a[u] = a[u + 1];
        if constexpr (!UNIT) w[u] = w[u + 1];
      }
      a[D - 1] = ix[D * 64 + l];
      ix += 64;
      if constexpr (UNIT) {
        sum += pi - v0;
        sum += pi - v1;
      } else {
        w[D - 1] = wx[D * 64 + l];
        wx += 64;
        sum += w0.x * (pi - v0);
        sum += w0.y * (pi - v1);
      }
    }
    return sum;
  }
};

// The wave's slice offsets, slot j's in lane j.
__device__ __forceinline__ int col_first(const ColGraph& g) {
  const int slots = g.slots + g.vslots;
  return g.soff[wave_here() * slots + min((int)(threadIdx.x & 63), slots)];
}

// The parts of heavy rows a thread walks and, where it owns a heavy row, that
// row's parts: the same in every apply, so read once.
struct ColParts {
  int own[2];    // heavy row of the thread's part in each further slot
  int lo, hi;    // parts of heavy row threadIdx.x
  __device__ __forceinline__ explicit ColParts(const ColGraph& g) : own{0, 0}, lo(0), hi(0) {
    const int t = threadIdx.x;
    if (g.vslots > 0) own[0] = g.vown[t];
    if (g.vslots > 1) own[1] = g.vown[t + kColBS];
    if (t < g.nh) {
      lo = g.voff[t];
      hi = g.voff[t + 1];
    }
  }
  // Sums of the parts (the stream's last slots) to hq; returns this thread's
  // share of sum p_i (L p)_i.
  // With PART: p holds positions [base, base + count), the row's own value
  // comes from `mine`, and the sums are added to hq from the second part on.
  template <typename V, bool UNIT, bool PART = false>
  __device__ __forceinline__ double walk(const ColGraph& g, ColStream<V, UNIT>& st, int first, const V* p,
                                         double* hq, const V* mine = nullptr, unsigned base = 0,
                                         unsigned count = 0) const {
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j < g.vslots) {
        const int v = threadIdx.x + j * kColBS;
        const V pi = PART ? mine[own[j]] : p[own[j]];
        double q = (double)st.template row<PART>(first, g.slots + j, p, pi, base, count);
        if (PART && base > 0 && v < g.nv) q += hq[v];
        if (v < g.nv) hq[v] = q;
        acc += (double)pi * q;
      }
    }
    return acc;
  }
  // Heavy row threadIdx.x from its parts.
  __device__ __forceinline__ double whole(const double* hq) const {
    double q = 0.0;
    for (int v = lo; v < hi; ++v) q += hq[v];
    return q;
  }
};

// How a CG run ended.
struct ColRun {
  int iters;      // iterations of this run
  int status;     // kStOk, kStNoconv, kStBreak
};

// Element t + 1024 j of a vector in memory: the slot in the (scalar) base,
// the thread in one 32-bit byte offset that all slots share.
template <typename V>
__device__ __forceinline__ V* slot_at(V* v, int j, int t) {
  return reinterpret_cast<V*>(
      reinterpret_cast<char*>(const_cast<typename std::remove_const<V>::type*>(v) + j * kColBS) +
      (unsigned)(t * (int)sizeof(V)));
}

// CG with the Jacobi preconditioner from residual rv and x (in memory),
// p = D^-1 r at the start, rho = r^T D^-1 r: iterations until ||r||^2 <=
// tol2 * bnorm2.  p lives in LDS, r and q in registers, x and 1/degree in
// registers where they suffice.  Three barriers an iteration: the sums of
// p^T q, of r^T z and r^T r, and the new p before it is gathered.  Vectors
// reach to the end of the last slot and are zero past n, so that no element
// is tested: at n = 10^4 an iteration is bound by the instructions of its
// 160 (wave, slot) steps.
template <typename V, bool UNIT, int EPT>
__device__ __forceinline__ ColRun col_cg(const ColGraph& g, V* p, double* hq, V (&rv)[EPT], V* x,
                                         double rho, double bnorm2, double tol2, int max_iter,
                                         ColShared& S, int& turn) {
  constexpr bool kXReg = EPT * sizeof(V) <= 40;
  constexpr bool kIReg = EPT * sizeof(V) <= 40;
  int t = thread_here();
  const V* inv = ColW<V>::inv(g);
  V qv[EPT], xv[kXReg ? EPT : 1], iv[kIReg ? EPT : 1];
#pragma unroll
  for (int j = 0; j < EPT; ++j) {
    if (j < g.slots) {
      if constexpr (kXReg) xv[j] = *slot_at(x, j, t);
      const V id = *slot_at(inv, j, t);
      if constexpr (kIReg) iv[j] = id;
      p[t + j * kColBS] = rv[j] * id;
    }
    four_at_a_time<EPT>(j);
  }
  const int first = col_first(g);
  const ColParts parts(g);
  constexpr bool kKeep = EPT <= 2;   // the stream's first rows stay in registers
  ColStream<V, UNIT> st;
  if constexpr (kKeep) st.start(g, first);
  ColRun run{0, kStOk};
  __syncthreads();
  for (;;) {
    t = thread_here();
    double dot[1] = {0.0};
    ColStream<V, UNIT> su;
    if constexpr (kKeep) su = st; else su.start(g, first);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        const V pi = p[t + j * kColBS];
        qv[j] = su.row(first, j, p, pi);
        // (a heavy row's own sum is 0 here: its product is that of its parts)
        dot[0] += (double)pi * (double)qv[j];
      }
      if (EPT > 1) asm volatile("" ::: "memory");
    }
    if (g.vslots > 0) dot[0] += parts.template walk<V, UNIT>(g, su, first, p, hq);
    col_sum<1>(dot, S, turn);
    if (uniform(!(dot[0] > 0.0) || !isfinite(dot[0]))) {
      run.status = kStBreak;
      break;
    }
    const V al = (V)(rho / dot[0]);
    double rr[2] = {0.0, 0.0};
    t = thread_here();
    if (parts.hi > 0) qv[0] = (V)parts.whole(hq);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        const V pi = p[t + j * kColBS];
        if constexpr (kXReg)
          xv[j] += al * pi;
        else
          *slot_at(x, j, t) += al * pi;
        rv[j] -= al * qv[j];
        const double rd = (double)rv[j];
        V id;
        if constexpr (kIReg) id = iv[j]; else id = *slot_at(inv, j, t);
        rr[0] += rd * rd * (double)id;
        rr[1] += rd * rd;
        qv[j] = rv[j] * id;   // q is done with: z for the direction
      }
      four_at_a_time<EPT>(j);
    }
    col_sum<2>(rr, S, turn);
    run.iters += 1;
    if (uniform(rr[1] <= tol2 * bnorm2)) break;
    if (run.iters >= max_iter) {
      run.status = kStNoconv;
      break;
    }
    if (uniform(!(rr[0] > 0.0) || !isfinite(rr[0]))) {
      run.status = kStBreak;
      break;
    }
    const V be = (V)(rr[0] / rho);
    rho = rr[0];
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        p[t + j * kColBS] = qv[j] + be * p[t + j * kColBS];
      }
      four_at_a_time<EPT>(j);
    }
    __syncthreads();
  }
  if constexpr (kXReg) {
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j)
      if (j < g.slots) *slot_at(x, j, t) = xv[j];
  }
  __syncthreads();
  return run;
}

// Means of v (memory, written and synchronised) over every component: the
// one mean of a connected graph is returned, several go to cm.  Components
// come largest first: the first by the block, the next by a wave each, the
// rest by a thread each.
__device__ __forceinline__ double col_means(const ColGraph& g, const double* v, double* cm, ColShared& S,
                                            int& turn) {
  const int t = threadIdx.x;
  if (g.nc == 1) {
    double a[1] = {0.0};
    for (int e = t; e < g.n; e += kColBS) a[0] += v[e];
    col_sum<1>(a, S, turn);
    return a[0] / (double)g.n;
  }
  for (int c = 0; c < g.nc_block; ++c) {
    const int lo = g.coff[c], hi = g.coff[c + 1];
    double a[1] = {0.0};
    for (int j = lo + t; j < hi; j += kColBS) a[0] += v[g.cnode[j]];
    col_sum<1>(a, S, turn);
    if (t == 0) cm[c] = a[0] / (double)(hi - lo);
  }
  for (int c = g.nc_block + (t >> 6); c < g.nc_wave; c += kColWaves) {
    const int lo = g.coff[c], hi = g.coff[c + 1];
    double a = 0.0;
    for (int j = lo + (t & 63); j < hi; j += 64) a += v[g.cnode[j]];
    a = wave_total(a);
    if ((t & 63) == 0) cm[c] = a / (double)(hi - lo);
  }
  for (int c = g.nc_wave + t; c < g.nc; c += kColBS) {
    const int lo = g.coff[c], hi = g.coff[c + 1];
    double a = 0.0;
    for (int j = lo; j < hi; ++j) a += v[g.cnode[j]];
    cm[c] = a / (double)(hi - lo);
  }
  __syncthreads();
  return 0.0;
}

__device__ __forceinline__ double col_mean(const ColGraph& g, const double* cm, double m, int e) {
  return g.nc == 1 ? m : cm[g.ccomp[e]];
}

// r = b - L x in FP64 (x, b, r in memory).  x is staged in LDS, whole or,
// where it does not fit, in two parts that are gathered from in turn (from
// memory the gathers of n = 3 10^4 took ten times as long).
template <bool UNIT>
__device__ __forceinline__ void col_resid(const ColGraph& g, const double* x, const double* b, double* r,
                                          double* lds, int lds_n, double* hq) {
  const int t = threadIdx.x;
  const int npad = g.slots * kColBS;
  const int first = col_first(g);
  const ColParts parts(g);
  __syncthreads();
  if (npad <= lds_n) {
    for (int e = t; e < npad; e += kColBS) lds[e] = x[e];
    __syncthreads();
    ColStream<double, UNIT> st;
    st.start(g, first);
    for (int j = 0; j < g.slots; ++j) {
      const int e = t + j * kColBS;
      const double y = st.row(first, j, lds, lds[e]);
      if (e < g.n) r[e] = b[e] - y;
    }
    if (g.vslots > 0) (void)parts.template walk<double, UNIT>(g, st, first, lds, hq);
  } else {
    for (int base = 0; base < npad; base += lds_n) {
      const int count = min(lds_n, npad - base);
      for (int e = t; e < count; e += kColBS) lds[e] = x[base + e];
      __syncthreads();
      ColStream<double, UNIT> st;
      st.start(g, first);
      for (int j = 0; j < g.slots; ++j) {
        const int e = t + j * kColBS;
        const double y = st.template row<true>(first, j, lds, x[e], base, count);
        if (e < g.n) r[e] = (base > 0 ? r[e] : b[e]) - y;
      }
      if (g.vslots > 0)
        (void)parts.template walk<double, UNIT, true>(g, st, first, lds, hq, x, base, count);
      __syncthreads();
    }
  }
  __syncthreads();
  if (t < g.nh) r[t] = b[t] - parts.whole(hq);
  __syncthreads();
}

}  // namespace nvd
