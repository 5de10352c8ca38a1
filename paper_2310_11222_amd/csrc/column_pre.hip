// The spanning forest and the approximate Cholesky factor in the order in
// which the one-block-per-column solver walks them, and its launches with
// either.
//
// On the multi-kernel path one application of the factor is a launch per
// elimination round and direction (n = 10^4: some 200 launches of ~3 us, 16 ms
// per 8 pairs), and one of the forest eight launches and three for its
// augmentation.  In one block a round is a barrier, and the forest's scans
// run over LDS.
#include <algorithm>
#include <cstring>
#include <vector>

#include "column_kernel.hpp"

namespace nvd {

namespace {

struct PreBlob {
  std::vector<unsigned char> h;
  template <typename T>
  size_t put(const std::vector<T>& v) {
    const size_t at = (h.size() + 255) & ~(size_t)255;
    h.resize(at + std::max<size_t>(sizeof(T) * v.size(), 1));
    if (!v.empty()) std::memcpy(h.data() + at, v.data(), sizeof(T) * v.size());
    return at;
  }
};

// One direction of the factor: rounds of positions (in the order they are
// taken), the pull list of each position.
struct Steps {
  std::vector<int4> steps;
  std::vector<unsigned short> idx;
  std::vector<double> c;
};

}  // namespace

// Rows of entries of a step: two, then as many fours as its longest list needs.
static int padded_rows(int longest, int gs) {
  const int rows = (longest + (1 << gs) - 1) >> gs;
  return rows <= 2 ? 2 : 2 + (rows - 2 + 3) / 4 * 4;
}

// Lanes per vertex of a round of m vertices whose longest list has `most`
// entries: the power of two with the least estimated time, in units of a step
// whose entries were read ahead; four further rows cost a read from L2, about
// another, and a reduction level a tenth.
static int lanes_log2(int m, int most) {
  int best = 0;
  double least = 1e300;
  for (int gs = 0; gs <= 6; ++gs) {
    const double passes = std::ceil((double)m * (1 << gs) / kColBS);
    const double t = passes * (1.0 + (padded_rows(most, gs) - 2) / 4.0 + 0.1 * gs);
    if (t < least) {
      least = t;
      best = gs;
    }
  }
  return best;
}

template <typename List>
static void add_round(Steps* st, int p0, int p1, bool always, const List& list) {
  int most = 0;
  for (int p = p0; p < p1; ++p) most = std::max(most, list(p).second);
  if (p1 <= p0 || (most == 0 && !always)) return;
  const int gs = most > 0 ? lanes_log2(p1 - p0, most) : 0;
  const int per = kColBS >> gs;
  for (int p = p0; p < p1; p += per) {
    const int m = std::min(per, p1 - p);
    int longest = 0;
    for (int i = 0; i < m; ++i) longest = std::max(longest, list(p + i).second);
    const int rows = padded_rows(longest, gs);
    const int width = m << gs;
    const int at = (int)st->idx.size();
    st->idx.resize(at + (size_t)rows * width, 0);
    st->c.resize(at + (size_t)rows * width, 0.0);
    for (int i = 0; i < m; ++i) {
      const auto l = list(p + i);
      for (int e = 0; e < l.second; ++e) {
        const size_t to = at + (size_t)(e >> gs) * width + (i << gs) + (e & ((1 << gs) - 1));
        st->idx[to] = l.first.first[e];
        st->c[to] = l.first.second[e];
      }
    }
    const bool last = p + m >= p1;
    st->steps.push_back(make_int4(p, m | gs << 12 | (last ? 1 << 16 : 0), rows, at));
  }
}

// The device layout of a preconditioner (its arrays are in one allocation).
struct ColPreDev {
  unsigned char* blob = nullptr;
  ColPre d{};
};

void free_column_pre(ColPreDev* p) {
  if (!p) return;
  (void)hipFree(p->blob);
  delete p;
}

static nvd_status upload(PreBlob& bl, ColPreDev** out, int64_t* bytes) {
  ColPreDev* cp = new ColPreDev();
  hipError_t e = device_alloc((void**)&cp->blob, bl.h.size());
  if (e == hipSuccess) e = hipMemcpy(cp->blob, bl.h.data(), bl.h.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    free_column_pre(cp);
    set_error(std::string("column preconditioner: ") + hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? NVD_E_NOMEM : NVD_E_DEVICE;
  }
  *bytes += (int64_t)bl.h.size();
  *out = cp;
  return NVD_OK;
}

static nvd_status build_achol(DevGraph* g, const std::vector<int>& perm, ColPreDev** out) {
  AcholPre* ap = g->achol;
  const int n = g->n;
  const size_t nf = (size_t)ap->nnz;
  // the factor as it is on the device, by elimination position
  std::vector<int> order(n), off[2], idx[2];
  std::vector<double> c[2], ip(n);
  hipError_t e = hipMemcpy(order.data(), ap->order, sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(ip.data(), ap->ip64, sizeof(double) * n, hipMemcpyDeviceToHost);
  for (int d = 0; d < 2; ++d) {
    off[d].resize(n + 1);
    idx[d].resize(nf);
    c[d].resize(nf);
    if (e == hipSuccess)
      e = hipMemcpy(off[d].data(), d ? ap->out_off : ap->in_off, sizeof(int) * (n + 1), hipMemcpyDeviceToHost);
    if (e == hipSuccess && nf)
      e = hipMemcpy(idx[d].data(), d ? ap->out_idx : ap->in_idx, sizeof(int) * nf, hipMemcpyDeviceToHost);
    if (e == hipSuccess && nf)
      e = hipMemcpy(c[d].data(), d ? ap->out_c64 : ap->in_c64, sizeof(double) * nf, hipMemcpyDeviceToHost);
  }
  if (e != hipSuccess) {
    set_error(std::string("column preconditioner: ") + hipGetErrorString(e));
    return NVD_E_DEVICE;
  }
  std::vector<int> place(n);
  for (int p = 0; p < n; ++p) place[order[p]] = p;
  std::vector<unsigned short> apos(n);
  for (int i = 0; i < n; ++i) apos[i] = (unsigned short)place[perm[i]];
  const int rounds = (int)ap->round_off.size() - 1;
  PreBlob bl;
  size_t o_steps[2], o_idx[2], o_c64[2], o_c32[2];
  int nsteps[2];
  for (int d = 0; d < 2; ++d) {
    std::vector<unsigned short> at(nf);
    for (size_t i = 0; i < nf; ++i) at[i] = (unsigned short)place[idx[d][i]];
    Steps st;
    auto list = [&](int p) {
      return std::make_pair(std::make_pair(at.data() + off[d][p], c[d].data() + off[d][p]),
                            off[d][p + 1] - off[d][p]);
    };
    for (int k = 0; k < rounds; ++k) {
      const int r = d ? rounds - 1 - k : k;
      add_round(&st, ap->round_off[r], ap->round_off[r + 1], d == 1, list);
    }
    nsteps[d] = (int)st.steps.size();
    st.steps.push_back(make_int4(0, 0, 0, 0));
    st.steps.push_back(make_int4(0, 0, 0, 0));
    std::vector<float> c32(st.c.begin(), st.c.end());
    o_steps[d] = bl.put(st.steps);
    o_idx[d] = bl.put(st.idx);
    o_c64[d] = bl.put(st.c);
    o_c32[d] = bl.put(c32);
  }
  std::vector<float> ip32(ip.begin(), ip.end());
  const size_t o_apos = bl.put(apos), o_ip64 = bl.put(ip), o_ip32 = bl.put(ip32);
  ColPreDev* cp = nullptr;
  NVD_TRY(upload(bl, &cp, &ap->bytes));
  g->bytes += (int64_t)bl.h.size();
  cp->d.kind = kColPreAchol;
  cp->d.apos = reinterpret_cast<const unsigned short*>(cp->blob + o_apos);
  cp->d.ip64 = reinterpret_cast<const double*>(cp->blob + o_ip64);
  cp->d.ip32 = reinterpret_cast<const float*>(cp->blob + o_ip32);
  for (int d = 0; d < 2; ++d) {
    cp->d.steps[d] = reinterpret_cast<const int4*>(cp->blob + o_steps[d]);
    cp->d.nsteps[d] = nsteps[d];
    cp->d.idx[d] = reinterpret_cast<const unsigned short*>(cp->blob + o_idx[d]);
    cp->d.c64[d] = reinterpret_cast<const double*>(cp->blob + o_c64[d]);
    cp->d.c32[d] = reinterpret_cast<const float*>(cp->blob + o_c32[d]);
  }
  *out = cp;
  return NVD_OK;
}

static nvd_status build_tree_order(DevGraph* g, const std::vector<int>& perm, int slots, ColPreDev** out) {
  TreePre* tp = g->tree;
  const int n = g->n, k = tp->k_aug;
  std::vector<int> tin(n), tout(n), rbeg(n), rend(n), tnode(2 * (size_t)n), uv(2 * (size_t)k);
  std::vector<double> winv(n), Cinv((size_t)k * k);
  hipError_t e = hipMemcpy(tin.data(), tp->tin, sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(tout.data(), tp->tout, sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(rbeg.data(), tp->rbeg, sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(rend.data(), tp->rend, sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(winv.data(), tp->winv, sizeof(double) * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess && k) e = hipMemcpy(uv.data(), tp->aug_uv, sizeof(int) * uv.size(), hipMemcpyDeviceToHost);
  if (e == hipSuccess && k)
    e = hipMemcpy(Cinv.data(), tp->aug_Cinv, sizeof(double) * Cinv.size(), hipMemcpyDeviceToHost);
  if (e != hipSuccess) {
    set_error(std::string("column preconditioner: ") + hipGetErrorString(e));
    return NVD_E_DEVICE;
  }
  // preorder places: entries counted along the tour
  std::vector<int> pre(n), at(2 * (size_t)n, -1), left(2 * (size_t)n, -1);
  for (int v = 0; v < n; ++v) {
    at[tin[v]] = v;
    left[tout[v]] = v;
  }
  const int per = 2 * slots;
  std::vector<unsigned short> tour((size_t)per * kColBS, (unsigned short)kColNoEvent);
  int entered = 0;
  for (int i = 0; i < 2 * n; ++i) {
    const size_t to = (size_t)(i % per) * kColBS + i / per;
    if (at[i] >= 0) {
      pre[at[i]] = entered;
      tour[to] = (unsigned short)entered;
      ++entered;
    } else {
      tour[to] = (unsigned short)(pre[left[i]] | 0x8000);
    }
  }
  std::vector<unsigned short> tpre(n), tsize(n), tlo(n), thi(n);
  std::vector<double> tw(n);
  for (int i = 0; i < n; ++i) {
    const int v = perm[i];
    tpre[i] = (unsigned short)pre[v];
    tsize[i] = (unsigned short)((tout[v] - tin[v] + 1) / 2);
    tlo[i] = (unsigned short)(rbeg[v] / 2);           // whole components come before
    thi[i] = (unsigned short)(rend[v] / 2);
    tw[i] = winv[v];
  }
  // the nodes that augmenting edges touch, each with its edges
  std::vector<unsigned short> auv(2 * (size_t)k), aend, aedge;
  std::vector<int> aoff(1, 0);
  std::vector<std::pair<int, int>> ends;
  for (int i = 0; i < k; ++i) {
    auv[i] = (unsigned short)pre[uv[i]];
    auv[k + i] = (unsigned short)pre[uv[k + i]];
    ends.push_back({auv[i], i});
    ends.push_back({auv[k + i], i | 0x8000});
  }
  std::sort(ends.begin(), ends.end());
  for (size_t i = 0; i < ends.size(); ++i) {
    if (i == 0 || ends[i].first != ends[i - 1].first) {
      if (i > 0) aoff.push_back((int)i);
      aend.push_back((unsigned short)ends[i].first);
    }
    aedge.push_back((unsigned short)ends[i].second);
  }
  if (!ends.empty()) aoff.push_back((int)ends.size());
  PreBlob bl;
  const size_t o_pre = bl.put(tpre), o_size = bl.put(tsize), o_lo = bl.put(tlo), o_hi = bl.put(thi);
  const size_t o_w = bl.put(tw), o_tour = bl.put(tour), o_auv = bl.put(auv), o_C = bl.put(Cinv);
  const size_t o_aoff = bl.put(aoff), o_aend = bl.put(aend), o_aedge = bl.put(aedge);
  ColPreDev* cp = nullptr;
  NVD_TRY(upload(bl, &cp, &tp->col_bytes));
  g->bytes += tp->col_bytes;
  auto us = [&](size_t o) { return reinterpret_cast<const unsigned short*>(cp->blob + o); };
  cp->d.kind = kColPreTree;
  cp->d.tpre = us(o_pre);
  cp->d.tsize = us(o_size);
  cp->d.tlo = us(o_lo);
  cp->d.thi = us(o_hi);
  cp->d.twinv = reinterpret_cast<const double*>(cp->blob + o_w);
  cp->d.tour = us(o_tour);
  cp->d.k = k;
  cp->d.nend = (int)aend.size();
  cp->d.auv = us(o_auv);
  cp->d.Cinv = reinterpret_cast<const double*>(cp->blob + o_C);
  cp->d.aoff = reinterpret_cast<const int*>(cp->blob + o_aoff);
  cp->d.aend = us(o_aend);
  cp->d.aedge = us(o_aedge);
  *out = cp;
  return NVD_OK;
}

nvd_status ensure_column_pre(DevGraph* g, bool achol, const int* perm_dev, int slots, ColPre* out) {
  if (achol)
    NVD_TRY(ensure_achol(g));
  else
    NVD_TRY(ensure_tree(g, 8));   // (tiles of 8 build the augmentation's matrix)
  if (!achol && g->tree->k_aug > kColMaxAug) {
    set_error("column solve: too many augmenting edges");
    return NVD_E_UNSUPPORTED;
  }
  ColPreDev** keep = achol ? &g->achol->col : &g->tree->col;
  if (!*keep) {
    std::vector<int> perm(g->n);
    NVD_HIP(hipMemcpy(perm.data(), perm_dev, sizeof(int) * g->n, hipMemcpyDeviceToHost));
    NVD_TRY(achol ? build_achol(g, perm, keep) : build_tree_order(g, perm, slots, keep));
  }
  *out = (*keep)->d;
  return NVD_OK;
}

template <bool MIXED, bool UNIT>
static nvd_status launch_pre_n(const ColArgs& a, int n, int blocks, size_t bytes, hipStream_t s) {
  const int ept = (n + kColBS - 1) / kColBS;
  if (ept <= 2) return launch_column_k<MIXED, UNIT, 2, true>(a, blocks, bytes, s);
  if (ept <= 8) return launch_column_k<MIXED, UNIT, 8, true>(a, blocks, bytes, s);
  if constexpr (MIXED) {
    if (ept <= 18) return launch_column_k<MIXED, UNIT, 18, true>(a, blocks, bytes, s);
    return launch_column_k<MIXED, UNIT, kColMaxPreEPT, true>(a, blocks, bytes, s);
  } else {
    return launch_column_k<MIXED, UNIT, 17, true>(a, blocks, bytes, s);
  }
}

nvd_status launch_column_pre(const ColArgs& a, bool mixed, bool unit, int n, int blocks, size_t bytes,
                             hipStream_t s) {
  if (mixed)
    return unit ? launch_pre_n<true, true>(a, n, blocks, bytes, s)
                : launch_pre_n<true, false>(a, n, blocks, bytes, s);
  return unit ? launch_pre_n<false, true>(a, n, blocks, bytes, s)
              : launch_pre_n<false, false>(a, n, blocks, bytes, s);
}

}  // namespace nvd
