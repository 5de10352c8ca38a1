// Explicit preconditioners in the one-block-per-column solver: z = M^-1 r in
// the block, M the augmented spanning forest or the approximate Cholesky
// factor, and the CG loop around it.
#pragma once

#include "column_dev.hpp"

namespace nvd {

// Position (within its wave's step) of a pull list's entry: see achol_block.
struct ColStep {
  int p0;        // first elimination position of the step
  int shape;     // vertices | log2(lanes per vertex) << 12 | barrier after it << 16
  int rows;      // entries of each lane
  int at;        // first entry
};

__device__ __forceinline__ ColStep step_of(const int4& v) {
  return {__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
          __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w)};
}

// Sum over groups of 2^gs lanes (gs uniform): register moves within rows of
// 16 lanes, shuffles beyond.
__device__ __forceinline__ double group_sum(double v, int gs) {
  if (gs > 0) v += dpp_move<0xB1>(v);
  if (gs > 1) v += dpp_move<0x4E>(v);
  if (gs > 2) v += dpp_move<0x141>(v);
  if (gs > 3) v += dpp_move<0x140>(v);
  if (gs > 4) v += __shfl_xor(v, 16, 64);
  if (gs > 5) v += __shfl_xor(v, 32, 64);
  return v;
}

// One triangular solve of the factor, y in LDS by elimination position.  The
// factor's rounds come as steps of at most 1024 lanes, several lanes to a
// vertex where its round is narrow and its lists long, each lane's entries
// rows as wide as the step in memory; a barrier ends every round.  While a
// step runs, the first two entries (and the pivot) of the next one and the
// description of the one after are on their way: a round then costs a
// barrier and an LDS gather, not the launch it was.
template <typename V, bool BACK>
__device__ __forceinline__ void achol_block(const ColPre& q, V* y) {
  constexpr int D = BACK ? 1 : 0;
  const int t = threadIdx.x;
  const unsigned short* idx = q.idx[D];
  const V* cf = sizeof(V) == 8 ? (const V*)q.c64[D] : (const V*)q.c32[D];
  const V* ip = sizeof(V) == 8 ? (const V*)q.ip64 : (const V*)q.ip32;
  struct Ahead {
    unsigned i[2];
    V c[2], d;
  };
  // (every step has two rows of entries, zero ones if need be)
  auto fetch = [&](const ColStep& s, Ahead& f) {
    const int gs = (s.shape >> 12) & 7;
    const int width = (s.shape & 0xfff) << gs;
    f.i[0] = f.i[1] = 0;
    f.c[0] = f.c[1] = f.d = (V)0;
    if (t < width) {
      f.i[0] = idx[s.at + t];
      f.c[0] = cf[s.at + t];
      f.i[1] = idx[s.at + width + t];
      f.c[1] = cf[s.at + width + t];
      if constexpr (BACK) f.d = ip[s.p0 + (t >> gs)];
    }
  };
  ColStep cur = step_of(q.steps[D][0]);
  ColStep nxt = step_of(q.steps[D][1]);
  Ahead have;
  fetch(cur, have);
  for (int s = 0; s < q.nsteps[D]; ++s) {
    const int4 later = q.steps[D][s + 2];
    Ahead want;
    fetch(nxt, want);
    const int m = cur.shape & 0xfff, gs = (cur.shape >> 12) & 7;
    const int width = m << gs;
    const int p = cur.p0 + (t >> gs);
    double acc = 0.0;
    V own = (V)0;
    if (t < width) {
      own = y[p];
      acc = (double)have.c[0] * (double)y[have.i[0]] + (double)have.c[1] * (double)y[have.i[1]];
      for (int j = 2; j < cur.rows; j += 4) {   // (rows come in twos and then in fours)
        unsigned i[4];
        V c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          i[u] = idx[cur.at + (j + u) * width + t];
          c[u] = cf[cur.at + (j + u) * width + t];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += (double)c[u] * (double)y[i[u]];
      }
    }
    acc = group_sum(acc, gs);
    if (t < width && (t & ((1 << gs) - 1)) == 0)
      y[p] = BACK ? (V)((double)own * (double)have.d + acc) : (V)((double)own + acc);
    if (cur.shape >> 16) __syncthreads();
    cur = nxt;
    nxt = step_of(later);
    have = want;
  }
  __syncthreads();
}

// Exclusive prefix of one value per thread, in thread order.
__device__ __forceinline__ double col_prefix(double v, ColShared& S, int& turn) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  double inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double up = __shfl_up(inc, off, 64);
    if (lane >= off) inc += up;
  }
  const double up = __shfl_up(inc, 1, 64);
  if (lane == 63) S.part[turn][0][w] = inc;
  __syncthreads();
  double base = 0.0;
  for (int i = 0; i < w; ++i) base += S.part[turn][0][i];
  turn ^= 1;
  return base + (lane > 0 ? up : 0.0);
}

// z = L_T^+ E for the spanning forest, E in LDS by preorder position (zero
// past n), z to memory by preorder position: the subtree sums as differences
// of E's prefix, the edge flows over the weights, and the potentials as their
// running sum over the Euler tour (entered +, left -), which a thread takes
// 2 * slots events of.  y: scratch in memory.
__device__ __forceinline__ void tree_block(const ColGraph& g, const ColPre& q, double* E, double* z, double* y,
                                           ColShared& S, int& turn) {
  const int t = threadIdx.x;
  const int c = g.slots;
  __syncthreads();
  double sum = 0.0;
#pragma unroll 4
  for (int i = t * c; i < t * c + c; ++i) sum += E[i];
  double run = col_prefix(sum, S, turn);
#pragma unroll 4
  for (int i = t * c; i < t * c + c; ++i) {
    run += E[i];
    E[i] = run;
  }
  __syncthreads();
#pragma unroll 4
  for (int e = t; e < g.n; e += kColBS) {
    const int a = q.tpre[e], size = q.tsize[e], lo = q.tlo[e], hi = q.thi[e];
    const double whole = E[hi] - (lo > 0 ? E[lo - 1] : 0.0);
    const double mu = whole / (double)(hi - lo + 1);
    const double f = E[a + size - 1] - (a > 0 ? E[a - 1] : 0.0) - mu * (double)size;
    y[a] = f * q.twinv[e];
  }
  __syncthreads();
#pragma unroll 4
  for (int i = t; i < c * kColBS; i += kColBS) E[i] = i < g.n ? y[i] : 0.0;
  __syncthreads();
  // (an event that is none reads some value of E and adds zero of it: the
  // loads of several events stay in flight together)
  const int last = c * kColBS - 1;
  sum = 0.0;
#pragma unroll 4
  for (int j = 0; j < 2 * c; ++j) {
    const int ev = q.tour[j * kColBS + t];
    const double v = E[min(ev & 0x7fff, last)];
    sum += ev == kColNoEvent ? 0.0 : (ev & 0x8000 ? -v : v);
  }
  run = col_prefix(sum, S, turn);
#pragma unroll 4
  for (int j = 0; j < 2 * c; ++j) {
    const int ev = q.tour[j * kColBS + t];
    const double v = E[min(ev & 0x7fff, last)];
    run += ev == kColNoEvent ? 0.0 : (ev & 0x8000 ? -v : v);
    if (ev < kColNoEvent) z[ev] = run;
  }
  __syncthreads();
}

constexpr int kColMaxAug = 256;                   // augmenting edges at most
constexpr int kColAugLds = 5 * kColMaxAug;        // values of LDS that takes

// The augmentation: z -= L_T^+ U C^-1 U^T z with a second forest solve in
// place of the n x k product (U's columns are the k edges, C^-1 is k x k).
// On return z2 holds what is to be subtracted.
__device__ __forceinline__ void tree_augment(const ColGraph& g, const ColPre& q, double* E, const double* z,
                                             double* z2, double* y, ColShared& S, int& turn) {
  const int t = threadIdx.x;
  const int k = q.k;
  double* s = E;                 // [256], then the four partial products [4][256]
  if (t < k) s[t] = z[q.auv[t]] - z[q.auv[k + t]];
  __syncthreads();
  // C^-1 is symmetric: thread (i, quarter of j) reads its columns side by side
  const int i = t & 255, part = t >> 8;
  double a = 0.0;
  if (i < k) {
    const int j0 = part * ((k + 3) / 4), j1 = min(k, j0 + (k + 3) / 4);
#pragma unroll 16
    for (int j = j0; j < j1; ++j) a += q.Cinv[(size_t)j * k + i] * s[j];
  }
  double* pr = E + 256;
  pr[part * 256 + i] = a;
  __syncthreads();
  double tv = 0.0;
  if (t < 256) tv = (pr[t] + pr[256 + t]) + (pr[512 + t] + pr[768 + t]);
  __syncthreads();
  // right-hand side U t: every end of an edge adds the edges it belongs to
  if (t < 256) y[t] = tv;
  for (int e = t; e < g.slots * kColBS; e += kColBS) E[e] = 0.0;
  __syncthreads();
  for (int v = t; v < q.nend; v += kColBS) {
    double sum = 0.0;
    for (int j = q.aoff[v]; j < q.aoff[v + 1]; ++j) {
      const unsigned ed = q.aedge[j];
      sum += ed & 0x8000u ? -y[ed & 0x7fffu] : y[ed];
    }
    E[q.aend[v]] = sum;
  }
  tree_block(g, q, E, z2, y, S, turn);
}

// z (in zv) = M^-1 r, r in rv; sum_r: the sum of r over the graph (used on
// connected graphs; else the component means go to cm).  Every thread's LDS
// reads of p must be behind a barrier.  work: four vectors.
template <typename V, int EPT>
__device__ __forceinline__ void pre_apply(const ColGraph& g, const ColPre& q, double* lds, const V (&rv)[EPT],
                                          V (&zv)[EPT], double* work, long stride, double sum_r, double* cm,
                                          ColShared& S, int& turn) {
  int t = thread_here();
  double* const w0 = work;
  double* const w1 = work + stride;
  double* const w2 = w1 + stride;
  if (q.kind == kColPreTree) {
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        const int e = t + j * kColBS;
        lds[e < g.n ? (int)q.tpre[e] : e] = (double)rv[j];
      }
      four_at_a_time<EPT>(j);
    }
    tree_block(g, q, lds, w0, w2, S, turn);
    if (q.k > 0) tree_augment(g, q, lds, w0, w1, w2, S, turn);
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = t + j * kColBS;
      zv[j] = (V)0;
      if (e < g.n) {
        const int a = q.tpre[e];
        zv[j] = (V)(q.k > 0 ? w0[a] - w1[a] : w0[a]);
      }
      four_at_a_time<EPT>(j);
    }
  } else {
    double mean = sum_r / (double)g.n;
    if (g.nc > 1) {
#pragma unroll
      for (int j = 0; j < EPT; ++j)
        if (j < g.slots) *slot_at(w2, j, t) = (double)rv[j];
      __syncthreads();
      mean = col_means(g, w2, cm, S, turn);
      t = thread_here();
    }
    V* y = reinterpret_cast<V*>(lds);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = t + j * kColBS;
      if (e < g.n) y[q.apos[e]] = (V)((double)rv[j] - col_mean(g, cm, mean, e));
      four_at_a_time<EPT>(j);
    }
    __syncthreads();
    achol_block<V, false>(q, y);
    achol_block<V, true>(q, y);
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = t + j * kColBS;
      zv[j] = e < g.n ? y[q.apos[e]] : (V)0;
      four_at_a_time<EPT>(j);
    }
  }
}

// CG with an explicit preconditioner solve, as col_cg; p_old waits in memory
// while the solve uses its LDS.  A column whose r^T z is no longer positive
// is at rounding level: it stops, and the true residual that follows decides.
template <typename V, bool UNIT, int EPT>
__device__ __forceinline__ ColRun col_cg_pre(const ColGraph& g, const ColPre& q, V* p, double* lds, double* hq,
                                             V (&rv)[EPT], V* x, double* work, long stride, double* cm,
                                             double bnorm2, double tol2, int max_iter, ColShared& S,
                                             int& turn) {
  ColRun run{0, kStOk};
  V* const pold = reinterpret_cast<V*>(work + 3 * stride);
  V qv[EPT];
  int t = thread_here();
  const int first = col_first(g);
  const ColParts parts(g);
  double rho = 0.0;
  double rr[2] = {0.0, 0.0};      // r^T r, sum r
#pragma unroll
  for (int j = 0; j < EPT; ++j)
    if (j < g.slots) rr[1] += (double)rv[j];
  col_sum<2>(rr, S, turn);
  for (;;) {
    pre_apply<V, EPT>(g, q, lds, rv, qv, work, stride, rr[1], cm, S, turn);
    double rz[1] = {0.0};
#pragma unroll
    for (int j = 0; j < EPT; ++j)
      if (j < g.slots) rz[0] += (double)rv[j] * (double)qv[j];
    col_sum<1>(rz, S, turn);
    if (run.iters > 0 && uniform(!isfinite(rz[0]))) {
      run.status = kStBreak;
      break;
    }
    if (!uniform(rz[0] > 0.0)) break;
    const V be = run.iters > 0 ? (V)(rz[0] / rho) : (V)0;
    rho = rz[0];
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        V pn = qv[j];
        if (run.iters > 0) pn += be * *slot_at(pold, j, t);
        p[t + j * kColBS] = pn;
      }
      four_at_a_time<EPT>(j);
    }
    __syncthreads();
    double dot[1] = {0.0};
    ColStream<V, UNIT> su;
    su.start(g, first);
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        const V pi = p[t + j * kColBS];
        qv[j] = su.row(first, j, p, pi);
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
    rr[0] = rr[1] = 0.0;
    t = thread_here();
    if (parts.hi > 0) qv[0] = (V)parts.whole(hq);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (j < g.slots) {
        const V pi = p[t + j * kColBS];
        *slot_at(x, j, t) += al * pi;
        *slot_at(pold, j, t) = pi;
        rv[j] -= al * qv[j];
        rr[0] += (double)rv[j] * (double)rv[j];
        rr[1] += (double)rv[j];
      }
      four_at_a_time<EPT>(j);
    }
    col_sum<2>(rr, S, turn);
    run.iters += 1;
    if (uniform(rr[0] <= tol2 * bnorm2)) break;
    if (run.iters >= max_iter) {
      run.status = kStNoconv;
      break;
    }
  }
  __syncthreads();
  return run;
}

}  // namespace nvd
