// The one-block-per-column kernel and its launch (column.hip: the Jacobi
// preconditioner; column_pre.hip: the spanning forest and the approximate
// Cholesky factor).
#pragma once

#include <string>

#include "column_pre_dev.hpp"

namespace nvd {

// LDS for the gathered vector and the heavy rows' sums (a CU has 160 KB;
// the block's partial sums are static).
constexpr int kColLds = 152 * 1024;
// Slots of the kernel with an explicit preconditioner (FP64: 17).
constexpr int kColMaxPreEPT = 24;
// Status of a pair between the mixed launch and the FP64 one (never returned).
constexpr int kColResume = -1;

template <bool MIXED, bool UNIT, int EPT, bool PRE>
__global__ __launch_bounds__(kColBS) void k_column(ColArgs a) {
  extern __shared__ double lds[];
  __shared__ ColShared S;
  int t = thread_here();
  int turn = 0;
  ColGraph g;
  ColJob job;
  if (a.jobs) {
    job = a.jobs[blockIdx.x];
    g = a.graphs[job.graph];
  } else {
    g = a.g;
    job.out = blockIdx.x;
    job.voff = a.col0 + blockIdx.x;
    job.ld = a.ld;
    job.xoff = job.voff;
    job.ldx = a.ldx;
  }
  make_scalar(g);
  const int n = g.n;
  double* const hq = lds;                       // [nv], ahead of the vector
  double* const buf = lds + ((g.nv + 1) & ~1);
  const long stride = a.jobs ? (long)g.slots * kColBS : a.stride;
  double* const b = a.vec + (a.jobs ? job.work : (long)blockIdx.x * a.vecs * stride);
  double* const x = b + stride;
  double* const r = x + stride;
  double* const work = r + 2 * stride;       // scratch of an explicit preconditioner
  double* const cm = a.cmean + (size_t)blockIdx.x * a.cstride;

  int status = kStOk, iters = 0, refine = 0, fb = 0;
  if (!MIXED && a.resume) {
    if (a.info[job.out].status != kColResume) return;
    iters = a.info[job.out].iters;
    refine = a.info[job.out].refine_steps;
    fb = 1;
  }
  double init[2] = {0.0, 0.0};
  double rv[MIXED ? 1 : EPT];
  if (!MIXED && a.resume) {
    // b and x are those of the mixed launch; r is the residual of x
    col_resid<UNIT>(g, x, b, r, buf, a.lds_n, hq);
    t = thread_here();
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = t + j * kColBS;
      if constexpr (!MIXED) rv[j] = 0.0;
      if (e < n) {
        const double v = r[e];
        init[0] += b[e] * b[e];
        init[1] += v * v * g.inv64[e];
        if constexpr (!MIXED) rv[j] = v;
      }
      four_at_a_time<EPT>(j);
    }
    col_sum<2>(init, S, turn);
  } else {
    // (a2) delta_bar = (P - Q) minus its mean on every component
    for (int e = t; e < g.slots * kColBS; e += kColBS) {
      double v = 0.0;
      if (e < n) {
        const long at = job.voff + (long)g.perm[e] * job.ld;
        v = a.P[at] - (a.Q ? a.Q[at] : 0.0);
      }
      b[e] = v;
      x[e] = 0.0;
      r[e] = 0.0;
    }
    __syncthreads();
    const double mean0 = col_means(g, b, cm, S, turn);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = t + j * kColBS;
      if constexpr (!MIXED) rv[j] = 0.0;
      if (e < n) {
        const double v = b[e] - col_mean(g, cm, mean0, e);
        b[e] = v;
        r[e] = v;
        init[0] += v * v;
        init[1] += v * v * g.inv64[e];
        if constexpr (!MIXED) rv[j] = v;
      }
      four_at_a_time<EPT>(j);
    }
    col_sum<2>(init, S, turn);
  }
  const double bb = init[0];
  double rho = init[1];
  int open = bb > 0.0;
  bool fp64_done = false;

  if constexpr (MIXED) {
    float* const x32 = reinterpret_cast<float*>(r + stride);
    float* const p32 = reinterpret_cast<float*>(buf);
    int stall = 0;
    double orr = bb;
    for (int step = 0; uniform(open != 0) && step <= a.max_refine; ++step) {
      double m = 0.0;
      if (step > 0) {
        // (a7) FP64 outer residual, projected
        col_resid<UNIT>(g, x, b, r, buf, a.lds_n, hq);
        m = col_means(g, r, cm, S, turn);
      }
      float f[EPT];
      t = thread_here();
      double s3[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < EPT; ++j) {
        const int e = t + j * kColBS;
        f[j] = 0.0f;
        if (j < g.slots) x32[e] = 0.0f;
        if (e < n) {
          const double v = r[e] - (step > 0 ? col_mean(g, cm, m, e) : 0.0);
          f[j] = (float)v;
          const float z = f[j] * g.inv32[e];
          s3[0] += v * v;
          s3[1] += (double)f[j] * (double)z;
          s3[2] += (double)f[j] * (double)f[j];
        }
        four_at_a_time<EPT>(j);
      }
      col_sum<3>(s3, S, turn);
      const double rr = s3[0];
      if (step > 0 && a.call) stall = refine_stall_count(orr, rr, stall, a.stall_ratio2);
      orr = rr;
      if (uniform(step > 0 && rr <= a.rtol2 * bb)) {
        open = 0;
        break;
      }
      if (uniform(refine_hand_to_fp64(stall))) {
        open = 0;
        fb = 1;
        break;
      }
      if (refine >= a.max_refine) {
        open = 0;
        status = kStNoconv;
        break;
      }
      if (!uniform(s3[2] > 0.0)) {
        open = 0;               // the residual rounds to zero in FP32
        break;
      }
      refine += 1;
      const double need2 = rr > 0.0 ? 0.09 * a.rtol2 * bb / rr : 0.0;
      const double it2 = need2 > a.irtol2 ? (need2 < 0.25 ? need2 : 0.25) : a.irtol2;
      ColRun run;
      if constexpr (PRE)
        run = col_cg_pre<float, UNIT, EPT>(g, a.pre, p32, buf, hq, f, x32, work, stride, cm, s3[2], it2,
                                           a.max_iter,
                                           S, turn);
      else
        run = col_cg<float, UNIT, EPT>(g, p32, hq, f, x32, s3[1], s3[2], it2, a.max_iter, S, turn);
      iters += run.iters;
      if (run.status == kStOk || (run.status == kStNoconv && !a.call)) {
        for (int e = t; e < n; e += kColBS) x[e] += (double)x32[e];
      } else {
        open = 0;
        if (run.status == kStNoconv)
          fb = 1;               // FP64 finishes from the last good x
        else
          status = run.status;
      }
    }
    if (fb) {
      // left to the FP64 launch, which takes b and x from vec
      if (t == 0) {
        nvd_pair_info pi{};
        pi.status = kColResume;
        pi.iters = iters;
        pi.refine_steps = refine;
        a.info[job.out] = pi;
      }
      return;
    }
    // the last residual is that of the final x, whose shift to mean zero
    // leaves L x as it is
    __syncthreads();
    const double mx = col_means(g, x, cm, S, turn);
    for (int e = t; e < n; e += kColBS) x[e] -= col_mean(g, cm, mx, e);
  } else {
    fp64_done = true;
    for (int restarts = 0; open; ++restarts) {
      if (uniform(rho > 0.0)) {
        ColRun run;
        if constexpr (PRE)
          run = col_cg_pre<double, UNIT, EPT>(g, a.pre, buf, buf, hq, rv, x, work, stride, cm, bb, a.rtol2,
                                              a.max_iter,
                                              S, turn);
        else
          run = col_cg<double, UNIT, EPT>(g, buf, hq, rv, x, rho, bb, a.rtol2, a.max_iter, S, turn);
        iters += run.iters;
        status = run.status == kStNoconv && a.call != kColOwn ? kStOk : run.status;
      }
      const double mx = col_means(g, x, cm, S, turn);
      for (int e = t; e < n; e += kColBS) x[e] -= col_mean(g, cm, mx, e);
      col_resid<UNIT>(g, x, b, r, buf, a.lds_n, hq);
      double s2[2] = {0.0, 0.0};
      t = thread_here();
#pragma unroll
      for (int j = 0; j < EPT; ++j) {
        const int e = t + j * kColBS;
        if (e < n) {
          rv[j] = r[e];
          s2[0] += rv[j] * rv[j];
          s2[1] += rv[j] * rv[j] * g.inv64[e];
        }
        four_at_a_time<EPT>(j);
      }
      col_sum<2>(s2, S, turn);
      rho = s2[1];
      open = status == kStOk && uniform(s2[0] > a.rtol2 * bb);
      if (restarts >= 2 || (restarts == 1 && a.call == kColBatchTwo)) break;
    }
  }

  // (a8) quadratic form, distance, per-pair info; x out
  double dots[3] = {0.0, 0.0, 0.0};
  for (int e = t; e < n; e += kColBS) {
    const double xe = x[e], re = r[e];
    dots[0] += b[e] * xe;
    dots[1] += xe * re;
    dots[2] += re * re;
    const long at = job.xoff + (long)g.perm[e] * job.ldx;
    if (a.X) a.X[at] = xe;
    if (a.B) a.B[at] = b[e];
    if (a.R) a.R[at] = re;
  }
  col_sum<3>(dots, S, turn);
  if (t == 0) {
    const double dsq = bb > 0.0 ? dots[0] + dots[1] : 0.0;
    if (fp64_done && status == kStOk && open) status = kStNoconv;
    const double d0 = dsq > 0.0 ? dsq : 0.0;
    if (a.d_out) a.d_out[a.col0 + job.out] = a.out_dsq ? d0 : sqrt(d0);
    nvd_pair_info pi;
    pi.status = status;
    pi.iters = iters;
    pi.refine_steps = refine;
    pi.flags = fb ? NVD_INFO_FP64_FALLBACK : 0;
    pi.rel_res = bb > 0.0 ? sqrt(dots[2] / bb) : 0.0;
    pi.dsq_plain = bb > 0.0 ? dots[0] : 0.0;
    pi.dsq = dsq;
    a.info[job.out] = pi;
  }
}

template <bool MIXED, bool UNIT, int EPT, bool PRE>
static nvd_status launch_column_k(const ColArgs& a, int blocks, size_t bytes, hipStream_t s) {
  const void* f = reinterpret_cast<const void*>(&k_column<MIXED, UNIT, EPT, PRE>);
  NVD_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kColLds));
  k_column<MIXED, UNIT, EPT, PRE><<<blocks, kColBS, bytes, s>>>(a);
  NVD_HIP(hipGetLastError());
  return NVD_OK;
}

// Launches of `blocks` columns of an n-node graph with `bytes` of LDS.
nvd_status launch_column_jacobi(const ColArgs& a, bool mixed, bool unit, int n, int blocks, size_t bytes,
                                hipStream_t s);
nvd_status launch_column_pre(const ColArgs& a, bool mixed, bool unit, int n, int blocks, size_t bytes,
                             hipStream_t s);
// The preconditioner's layout for the one-block solver (column_pre.hip): the
// graph's forest or factor, which must be set up, in the block's order.
nvd_status ensure_column_pre(DevGraph* g, bool achol, const int* perm_dev, int slots, ColPre* out);

}  // namespace nvd
