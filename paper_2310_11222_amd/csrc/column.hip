// One block per column: the whole solve of one pair on a graph of up to a few
// ten thousand nodes in one block of 1024 threads, whose CG direction lives
// in that CU's LDS.
//
// On such graphs an iteration of the multi-kernel path, or of the
// cooperative launch with its grid barriers, is bound by launches and by
// coherent round trips between XCDs (24-34 us at n = 10^4), not by its few
// hundred kilobytes.  A column that stays in one CU needs neither: its
// gathers are LDS reads, its sums are register moves between lanes and one
// block barrier, and the other columns run on other CUs at the same time.
// What it gives up is the sharing of the graph between columns; the
// neighbour lists are 16-bit positions, read from L2 by every block.
//
// Measured per call, host included (before: cooperative launch, or the
// multi-kernel path on several components): BA n = 10^3, one pair, FP64, 337
// -> 106 us (1.8 us an iteration on a lattice of that size, 2.7 with hubs;
// ~32 us around them); ER n = 10^4, average degree 4, 214 components, 8 pairs
// mixed, 2025 -> 403 us; WS n = 10^4 of degree 16, weighted, 5 pairs FP64,
// 2868 -> 1091 us.  At n = 10^4 an FP64 iteration of 19 us is bound by the LDS
// (a random 64-lane gather of 8 bytes takes ~8.4 cycles of the CU, 160K
// entries ~9 us) and by the vector work of ten elements a thread (~6 us).
//
// The arithmetic is that of the other paths (same recurrences, stopping and
// refinement rules, same edge-difference form of L x); sums have a fixed
// order, so results repeat bit for bit.
#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <thread>
#include <vector>

#include "column_kernel.hpp"

namespace nvd {

// Rows with more neighbours than this (and more than twice the mean) are
// heavy, and cut into parts of at least kColPart neighbours, so many that at
// most kColMaxParts are needed.
constexpr int kColHeavyDeg = 16;
constexpr int kColPart = 16;
constexpr int kColMaxParts = 2048;
// Rows of more neighbours than this count as hubs in the choice of solver.
constexpr int kColHubDeg = 64;
constexpr int kColMaxEPT = 32;   // FP64: 17, what LDS holds
// Columns of one launch (one CU each).
constexpr int kColChunk = 256;
// Weights and 1 / degree in the block's order, from the graph's.
__global__ void k_column_weights(int entries, const int* src, int n, int npad, const int* perm,
                                 const double* w64, const double* invd64, const float* invd32, double* sw64,
                                 float* sw32, double* inv64, float* inv32) {
  const int step = gridDim.x * blockDim.x;
  const int i0 = blockIdx.x * blockDim.x + threadIdx.x;
  if (w64) {
    for (int i = i0; i < entries; i += step) {
      const double w = src[i] >= 0 ? w64[src[i]] : 0.0;
      sw64[i] = w;
      sw32[i] = (float)w;
    }
  }
  for (int i = i0; i < npad; i += step) {
    inv64[i] = i < n ? invd64[perm[i]] : 0.0;
    inv32[i] = i < n ? invd32[perm[i]] : 0.0f;
  }
}

// x of one column, by node (for the multi-kernel solver).
__global__ void k_column_nodes(int n, const int* perm, const double* x, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[perm[i]] = x[i];
}
__global__ void k_column_put(int n, const double* x, double* X, long ldx) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) X[(long)i * ldx] = x[i];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct ColPlan {
  ColGraph d{};
  unsigned char* blob = nullptr;   // what the host laid out
  double* weights = nullptr;       // what k_column_weights fills
  const int* src = nullptr;
  int entries = 0;
  bool weighted = false;           // the copies are those of explicit weights
  bool stale = true;               // the graph's weights changed since
  int64_t bytes = 0;               // of both
  int64_t weight_bytes = 0;
};

// Scratch (`vec` doubles of vectors, then `cm` of component means) and result
// words of a call, kept with the graph or the batch.
nvd_status ensure_column_ws(ColWs* w, size_t vec, size_t cm, int cols, int64_t* bytes) {
  if (w->cap_vec < vec || w->cap_cm < cm) {
    (void)hipFree(w->vec);
    w->vec = nullptr;
    if (bytes) *bytes -= (int64_t)(sizeof(double) * (w->cap_vec + w->cap_cm));
    w->cap_vec = w->cap_cm = 0;
    NVD_HIP(device_alloc((void**)&w->vec, sizeof(double) * (vec + cm)));
    w->cap_vec = vec;
    w->cap_cm = cm;
    if (bytes) *bytes += (int64_t)(sizeof(double) * (vec + cm));
  }
  if (w->cap_info < cols) {
    if (w->info) (void)hipHostFree(w->info);
    w->info = nullptr;
    w->cap_info = 0;
    const int c = std::max(cols, 64);
    const hipError_t e = hipHostMalloc((void**)&w->info, sizeof(nvd_pair_info) * c, hipHostMallocDefault);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      w->info = nullptr;
      set_error(std::string("hipHostMalloc: ") + hipGetErrorString(e));
      return NVD_E_NOMEM;
    }
    w->cap_info = c;
  }
  return NVD_OK;
}

void free_column_ws(ColWs* w) {
  if (w->vec) (void)hipFree(w->vec);
  if (w->info) (void)hipHostFree(w->info);
  *w = ColWs{};
}

void free_column(DevGraph* g) {
  if (g->col) {
    (void)hipFree(g->col->blob);
    (void)hipFree(g->col->weights);
    g->bytes -= g->col->bytes;
    delete g->col;
    g->col = nullptr;
  }
  if (g->col_ws.cap_vec) g->bytes -= (int64_t)(sizeof(double) * (g->col_ws.cap_vec + g->col_ws.cap_cm));
  free_column_ws(&g->col_ws);
}

void column_weights_changed(DevGraph* g) {
  if (g->col) g->col->stale = true;
}

namespace {

// Parts of one host buffer that becomes one device allocation.
struct Blob {
  std::vector<unsigned char> h;
  size_t put(const void* p, size_t bytes) {
    const size_t at = (h.size() + 255) & ~(size_t)255;
    h.resize(at + std::max<size_t>(bytes, 1));
    if (bytes) std::memcpy(h.data() + at, p, bytes);
    return at;
  }
};

}  // namespace

// The host's layout of a graph for the block (see ColGraph).
struct ColLayout {
  std::vector<int> perm, soff, src, voff, vown, coff, cnode, ccomp;
  std::vector<unsigned short> idx;
  ColGraph d{};                          // its counts
  // Appends the arrays to a buffer; the pointers of `d` become offsets in it.
  void put(Blob* bl);
  size_t o_src = 0;
};

static void layout_column(const DevGraph* g, ColLayout* lay) {
  const int n = g->n;
  const int* rp = g->h_rp.data();
  const int* ci = g->h_ci.data();
  // positions: nodes by falling degree, ties by node (counting sort)
  std::vector<int> first(g->max_deg + 2, 0), pos(n);
  std::vector<int>& perm = lay->perm;
  perm.resize(n);
  for (int i = 0; i < n; ++i) ++first[g->max_deg - (rp[i + 1] - rp[i]) + 1];
  std::partial_sum(first.begin(), first.end(), first.begin());
  for (int i = 0; i < n; ++i) {
    const int at = first[g->max_deg - (rp[i + 1] - rp[i])]++;
    perm[at] = i;
    pos[i] = at;
  }
  auto deg = [&](int e) { return rp[perm[e] + 1] - rp[perm[e]]; };
  const double heavy_at = std::max((double)kColHeavyDeg, 2.0 * g->nnz / n);
  int nh = 0;
  long hnnz = 0;
  while (nh < n && nh < kColBS && deg(nh) > heavy_at) hnnz += deg(nh++);
  int part = kColPart;
  while (hnnz / part + nh > kColMaxParts) part *= 2;
  std::vector<int>& voff = lay->voff;
  voff.assign(nh + 1, 0);
  for (int e = 0; e < nh; ++e) voff[e + 1] = voff[e] + (deg(e) + part - 1) / part;
  const int nv = voff[nh];
  const int slots = (n + kColBS - 1) / kColBS;
  const int vslots = (nv + kColBS - 1) / kColBS;
  std::vector<int>& vown = lay->vown;
  vown.assign(std::max(1, vslots * kColBS), 0);
  for (int e = 0; e < nh; ++e)
    for (int v = voff[e]; v < voff[e + 1]; ++v) vown[v] = e;
  // the neighbours of a lane's row: first entry, count, own position
  struct Row { int lo, count, own; };
  auto row_of = [&](int j, int w, int l) -> Row {
    if (j < slots) {
      const int e = j * kColBS + w * 64 + l;
      if (e < nh || e >= n) return {0, 0, e};
      return {rp[perm[e]], deg(e), e};
    }
    const int v = (j - slots) * kColBS + w * 64 + l;
    if (v >= nv) return {0, 0, 0};
    const int e = vown[v];
    const int lo = rp[perm[e]] + (v - voff[e]) * part;
    return {lo, std::min(part, rp[perm[e] + 1] - lo), e};
  };
  const int all = slots + vslots;
  std::vector<int>& soff = lay->soff;
  soff.assign(kColWaves * all + 1, 0);
  for (int w = 0; w < kColWaves; ++w)
    for (int j = 0; j < all; ++j) {
      int most = 0;
      for (int l = 0; l < 64; ++l) most = std::max(most, row_of(j, w, l).count);
      soff[w * all + j + 1] = soff[w * all + j] + (most + 1) / 2;
    }
  const size_t entries = (size_t)(soff[kColWaves * all] + kColSpare) * 128;
  std::vector<unsigned short>& idx = lay->idx;
  std::vector<int>& src = lay->src;
  idx.assign(entries, 0);
  src.assign(entries, -1);
  for (int w = 0; w < kColWaves; ++w)
    for (int j = 0; j < all; ++j) {
      const int at0 = soff[w * all + j], pairs = soff[w * all + j + 1] - at0;
      for (int l = 0; l < 64; ++l) {
        const Row r = row_of(j, w, l);
        for (int i = 0; i < 2 * pairs; ++i) {
          const size_t at = ((size_t)(at0 + i / 2) * 64 + l) * 2 + (i & 1);
          idx[at] = (unsigned short)(i < r.count ? pos[ci[r.lo + i]] : r.own);
          src[at] = i < r.count ? r.lo + i : -1;
        }
      }
    }
  // components, largest first
  const int nc = g->n_comp;
  std::vector<int>&coff = lay->coff, &cnode = lay->cnode, &ccomp = lay->ccomp;
  int nc_block = 0, nc_wave = 0;
  if (nc > 1) {
    std::vector<int> size(nc, 0), order(nc), rank(nc);
    for (int i = 0; i < n; ++i) ++size[g->h_comp[i]];
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return size[x] > size[y]; });
    coff.assign(nc + 1, 0);
    for (int c = 0; c < nc; ++c) {
      rank[order[c]] = c;
      coff[c + 1] = coff[c] + size[order[c]];
      if (size[order[c]] > 512) nc_block = c + 1;
      if (size[order[c]] > 16) nc_wave = c + 1;
    }
    cnode.resize(n);
    ccomp.resize(n);
    std::vector<int> at(coff.begin(), coff.end() - 1);
    for (int e = 0; e < n; ++e) {
      const int c = rank[g->h_comp[perm[e]]];
      ccomp[e] = c;
      cnode[at[c]++] = e;
    }
  }
  ColGraph& d = lay->d;
  d.n = n;
  d.nh = nh;
  d.nc = nc;
  d.slots = slots;
  d.vslots = vslots;
  d.nv = nv;
  d.nc_block = nc_block;
  d.nc_wave = std::max(nc_wave, nc_block);
}

void ColLayout::put(Blob* bl) {
  auto at = [&](const auto& v) {
    return bl->put(v.data(), sizeof(v[0]) * v.size());
  };
  // (offsets for now: `place` turns them into pointers)
  d.perm = reinterpret_cast<const int*>(at(perm));
  d.soff = reinterpret_cast<const int*>(at(soff));
  d.idx = reinterpret_cast<const unsigned*>(at(idx));
  o_src = at(src);
  d.voff = reinterpret_cast<const int*>(at(voff));
  d.vown = reinterpret_cast<const int*>(at(vown));
  d.coff = reinterpret_cast<const int*>(at(coff));
  d.cnode = reinterpret_cast<const int*>(at(cnode));
  d.ccomp = reinterpret_cast<const int*>(at(ccomp));
}

// Offsets of ColLayout::put as pointers into the device copy.
static ColGraph place(ColGraph d, const unsigned char* base) {
  auto fix = [&](auto& p) {
    p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + reinterpret_cast<size_t>(p));
  };
  fix(d.perm);
  fix(d.soff);
  fix(d.idx);
  fix(d.voff);
  fix(d.vown);
  fix(d.coff);
  fix(d.cnode);
  fix(d.ccomp);
  return d;
}

static nvd_status build_column(DevGraph* g) {
  ColLayout lay;
  layout_column(g, &lay);
  Blob bl;
  lay.put(&bl);
  ColPlan* cp = new ColPlan();
  hipError_t e = device_alloc((void**)&cp->blob, bl.h.size());
  if (e == hipSuccess) e = hipMemcpy(cp->blob, bl.h.data(), bl.h.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(cp->blob);
    delete cp;
    set_error(std::string("column plan: ") + hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? NVD_E_NOMEM : NVD_E_DEVICE;
  }
  cp->bytes = (int64_t)bl.h.size();
  cp->d = place(lay.d, cp->blob);
  cp->src = reinterpret_cast<const int*>(cp->blob + lay.o_src);
  cp->entries = (int)lay.src.size();
  g->col = cp;
  g->bytes += cp->bytes;
  return NVD_OK;
}

// Doubles that the weights and 1 / degrees of a layout take (FP64 and FP32).
static size_t weight_doubles(size_t entries, int npad) { return (12 * (entries + (size_t)npad) + 7) / 8; }

// Where they go: at `at` (weight_doubles of it), and filled from the graph's
// (w64 null: unit weights).
static nvd_status put_weights(const double* w64, const double* invd64, const float* invd32, ColGraph* d,
                              size_t entries, const int* src, double* at, hipStream_t s) {
  const int npad = d->slots * kColBS;
  const size_t sw = w64 ? entries : 0;
  float* f = reinterpret_cast<float*>(at + sw + npad);
  d->w64 = w64 ? reinterpret_cast<const double2*>(at) : nullptr;
  d->inv64 = at + sw;
  d->w32 = w64 ? reinterpret_cast<const float2*>(f) : nullptr;
  d->inv32 = f + sw;
  const int work = std::max((int)entries, npad);
  k_column_weights<<<std::min(1024, (work + 255) / 256), 256, 0, s>>>((int)entries, src, d->n, npad, d->perm, w64,
                                                                      invd64, invd32, at, f, at + sw, f + sw);
  NVD_HIP(hipGetLastError());
  return NVD_OK;
}

// The plan with the graph's present weights.
static nvd_status ensure_column(DevGraph* g, hipStream_t s) {
  if (!g->col) NVD_TRY(build_column(g));
  ColPlan* cp = g->col;
  if (!cp->stale) return NVD_OK;
  if (!cp->weights || cp->weighted != g->weighted) {
    (void)hipFree(cp->weights);
    cp->weights = nullptr;
    cp->bytes -= cp->weight_bytes;
    g->bytes -= cp->weight_bytes;
    cp->weight_bytes = 0;
    const size_t want = weight_doubles(g->weighted ? cp->entries : 0, cp->d.slots * kColBS);
    NVD_HIP(device_alloc((void**)&cp->weights, sizeof(double) * want));
    cp->weighted = g->weighted;
    cp->weight_bytes = (int64_t)(sizeof(double) * want);
    cp->bytes += cp->weight_bytes;
    g->bytes += cp->weight_bytes;
  }
  NVD_TRY(put_weights(g->weighted ? g->w64 : nullptr, g->invd64, g->invd32, &cp->d, cp->entries, cp->src,
                      cp->weights, s));
  cp->stale = false;
  return NVD_OK;
}

// Slots of the instantiations: the fewer, the fewer registers and elements past
// n.  Up to 8, powers of two (vectors wholly in registers).  Beyond, in mixed
// precision (us per 8 pairs, this instantiation / the next one kept: 18 for 10
// and 14, 33 for 24): 10 slots, the last with x and 1 / degree in registers, WS
// n = 10,000 738 / 1005, BA 285 / 342; 14 slots, WS n = 13,000 1068 / 1094, BA
// 366 / 379; 24 slots, WS n = 22,000 1875 / 1962, BA 710 / 732.
template <bool MIXED, bool UNIT>
static nvd_status launch_column_n(const ColArgs& a, int n, int blocks, size_t bytes, hipStream_t s) {
  const int ept = (n + kColBS - 1) / kColBS;
  if (ept <= 1) return launch_column_k<MIXED, UNIT, 1, false>(a, blocks, bytes, s);
  if (ept <= 2) return launch_column_k<MIXED, UNIT, 2, false>(a, blocks, bytes, s);
  if (ept <= 4) return launch_column_k<MIXED, UNIT, 4, false>(a, blocks, bytes, s);
  if (ept <= 8) return launch_column_k<MIXED, UNIT, 8, false>(a, blocks, bytes, s);
  if constexpr (MIXED) {
    if (ept <= 10) return launch_column_k<MIXED, UNIT, 10, false>(a, blocks, bytes, s);
    if (ept <= 14) return launch_column_k<MIXED, UNIT, 14, false>(a, blocks, bytes, s);
    if (ept <= 18) return launch_column_k<MIXED, UNIT, 18, false>(a, blocks, bytes, s);
    if (ept <= 24) return launch_column_k<MIXED, UNIT, 24, false>(a, blocks, bytes, s);
    // (33, one more than there are: arrays of 31 or 32 floats are kept as one
    // register tuple, which on weighted graphs was spilled as a whole, 4 KB a
    // thread: an iteration on 28,000 nodes of degree 8 took 252 us, now 28)
    return launch_column_k<MIXED, UNIT, 33, false>(a, blocks, bytes, s);
  } else {
    // (arrays of 9 to 16 doubles are kept as one register tuple each and
    // spill as a whole)
    return launch_column_k<MIXED, UNIT, 17, false>(a, blocks, bytes, s);
  }
}

nvd_status launch_column_jacobi(const ColArgs& a, bool mixed, bool unit, int n, int blocks, size_t bytes,
                                hipStream_t s) {
  if (mixed)
    return unit ? launch_column_n<true, true>(a, n, blocks, bytes, s)
                : launch_column_n<true, false>(a, n, blocks, bytes, s);
  return unit ? launch_column_n<false, true>(a, n, blocks, bytes, s)
              : launch_column_n<false, false>(a, n, blocks, bytes, s);
}

static size_t parts_bytes(int nv) { return sizeof(double) * (size_t)((nv + 1) & ~1); }

// Whether a column of n nodes fits one block: its elements in registers, its
// gathered vector (FP64, or FP32 in mixed precision) in LDS beside the most
// parts of heavy rows there can be.
static bool column_fits(int n, bool mixed) {
  const size_t npad = (size_t)(n + kColBS - 1) / kColBS * kColBS;
  return npad <= (size_t)kColBS * kColMaxEPT && npad * (mixed ? 4 : 8) + parts_bytes(kColMaxParts) <= (size_t)kColLds;
}

// Which solver takes k pairs of a graph that fits: the one with the smaller
// estimated time of a CG iteration, both fitted to measured times of 960 calls
// (BA, WS, ER, power law; n = 500 .. 3.2 10^4, average degree 4 to 64, unit and
// weighted, k = 1 .. 64, both precisions; half of them within 16%, nine in ten
// within 40%).  The faster one is taken but for 1% of the time in all, 4% of the
// calls being more than 5% slower than they could be.
//
// A block's iteration (us) grows with its slots (vector work) and with the
// graph's entries (LDS gathers), not with k: its columns run side by side.  The
// entries are read from the XCD's 4 MB L2 in every iteration, 2 bytes of index
// and the weight each; beyond it an entry costs two to three times as much,
// however many there are (n = 17,000 weighted, mixed, of degree 24: 46 us, of
// degree 48: 143; n = 6,000, unit, of degree 200: 71, of degree 500: 440).
static double stream_bytes(int nnz, bool weighted, bool fp64) {
  return (double)nnz * (weighted ? (fp64 ? 10.0 : 6.0) : 2.0);
}
static double block_iteration(int n, int nnz, int max_deg, bool weighted, bool fp64) {
  const double slots = (n + kColBS - 1) / kColBS;
  const double near = 6.0e-5 + (weighted ? 3.4e-5 : 0.0) + (max_deg > kColHubDeg ? 4.4e-5 : 0.0);
  const double beyond = std::min(1.0, std::max(0.0, (stream_bytes(nnz, weighted, fp64) - 3.5e6) / 2.0e6));
  return 2.6 + (fp64 ? 0.29 : 0.25) * slots + 3.6e-4 * std::max(0, n - 10 * kColBS) +
         nnz * (near + beyond * (1.9e-4 - near));
}

// An iteration of one tile of the other paths: the single launch (barriers, more
// with long rows and hubs, which its threads and waves walk), or the multi-kernel
// path (launches, one line per gather, and with several components their means).
static double tile_iteration(const DevGraph* g, int T, bool fp64) {
  const double n = g->n, nnz = g->nnz, nT = n * T, es = fp64 ? 8.0 : 4.0;
  const bool hubs = g->max_deg > kColHubDeg;
  if (g->n_comp == 1 && nT <= 524288.0)
    return (nT <= 2048.0 ? 2.5 : 8.0) + 0.67 * std::min(nnz / n, 40.0) + (hubs ? 14.0 : 0.0) + 7.0e-5 * nT +
           1.2e-7 * nnz * T;
  const double one = 29.0 + (hubs ? 18.0 : 0.0) + (1.5e-7 * nnz + 2.6e-6 * n) * T * es;
  return g->n_comp == 1 ? one : one - 7.0 + 1.4e-4 * g->max_comp * T;
}

// E.g. (us a call, block / tiles, mixed): ER n = 10^4 d = 4 k = 8 398 / 1975; WS
// n = 3.2 10^4 d = 8, weighted, k = 3 2246 / 2044, k = 48 2520 / 4801; BA n = 2.4
// 10^4 m = 8 k = 1 820 / 705; ER n = 1.7 10^4 d = 64, weighted, k = 7 2405 / 606.
static bool column_is_faster(const DevGraph* g, int k, const SolveParams& sp) {
  const bool fp64 = sp.precision != NVD_MIXED;
  const double block = block_iteration(g->n, g->nnz, g->max_deg, g->weighted, fp64);
  int tile = 1;                        // (not the timed one: results repeat)
  while (2 * tile <= std::min(k, 32)) tile *= 2;
  double tiles = 0.0;
  for (int left = k; left > 0;) {
    const int T = next_tile(g, k, left, tile, sp);
    tiles += tile_iteration(g, T, fp64);
    left -= T;
  }
  return block * ((k + kColChunk - 1) / kColChunk) <= tiles;
}

// The same with the forest: a block's iteration grows with its slots (two forest
// solves where there are off-forest edges to augment it with), that of tiles of up
// to eight pairs hardly with anything (us, block / tiles of 1, of 3 and of 8 pairs;
// BA m = 2 n = 11,000 mixed 83 / 121, 101, 107, n = 14,000 100 / 117, 97, 103, FP64
// 104 / 119, 94, 102, n = 17,000 114 / 119, 104, 114, FP64 119 / 120, 102, 112); of
// sixteen pairs 120 to 140, where the block still takes 114 (FP64 120).
static bool forest_is_faster(const DevGraph* g, int k, const SolveParams& sp) {
  const long off = (long)g->nnz / 2 - g->n + g->n_comp;
  if (k > 8 || off == 0) return true;
  const double slots = (g->n + kColBS - 1) / kColBS;
  const double block = 19.0 + (sp.precision == NVD_MIXED ? 5.7 : 6.1) * slots;
  return block <= (k == 1 ? 118.0 : (k <= 4 ? 98.0 : 103.0));
}

bool column_gives_way(DevGraph* g, nvd_status st) {
  if (st != NVD_E_UNSUPPORTED && st != NVD_E_NOMEM) return false;
  if (st == NVD_E_NOMEM) {
    free_column(g);
    g->col_failed = true;
  }
  set_error("");
  return true;
}

bool use_column(const DevGraph* g, int k, const SolveParams& sp) {
  if (sp.warm || g->col_failed) return false;
  if (sp.achol && g->n > kColBS * kColMaxPreEPT) return false;
  // (the forest's sums are FP64 in either precision)
  const bool fp64_vector = sp.precision != NVD_MIXED || (sp.tree && !sp.achol);
  if (!column_fits(g->n, !fp64_vector)) return false;
  // the switches of the other single-launch path ask for it, or for none
  const char* e = std::getenv("NVD_SMALL");
  if (e && e[0] == '0') return false;
  if (std::getenv("NVD_MID_BLOCKS")) return false;
  if (const char* c = std::getenv("NVD_COLUMN")) return c[0] != '0';   // 0 never, 1 wherever it fits
  // An explicit preconditioner costs the tiled path ten to hundreds of launches
  // an iteration.  The factor has two for every round (BA n = 10^4, 8 pairs, 16.5
  // ms; in blocks 2.0), and the block is taken wherever it fits: also on the
  // densest graphs measured (ER n = 14,000 of degree 32, 1.1M entries in the
  // factor, one pair, FP64) it took 16.0 ms against 27.9.
  if (sp.achol) return true;
  if (sp.tree) return forest_is_faster(g, k, sp);
  return column_is_faster(g, k, sp);
}

// A pair that FP32 cannot finish on a graph whose FP64 vector does not fit:
// the multi-kernel FP64 solver, from the pair's x.
static nvd_status finish_multi_kernel(DevGraph* g, int col, int block, const double* P, const double* Q,
                                      int64_t ld, const SolveParams& sp, const ColArgs& a,
                                      nvd_pair_info* info, hipStream_t s) {
  const int n = g->n;
  const double* x = a.vec + ((size_t)block * a.vecs + 1) * a.stride;
  double* X = const_cast<double*>(x) + a.stride;   // r's place
  k_column_nodes<<<(n + 255) / 256, 256, 0, s>>>(n, g->col->d.perm, x, X);
  NVD_HIP(hipGetLastError());
  SolveParams f = sp;
  f.precision = NVD_FP64;
  f.warm = true;
  f.cols = 1;
  NVD_TRY(ensure_workspace(g, 1, false));
  // (without a place for d: past the pair's x)
  double* d = a.d_out ? a.d_out + col : X + a.stride;
  NVD_TRY(solve_tile(g, 1, P + col, Q ? Q + col : nullptr, ld, f, d, X, 1, g->ws->info, s));
  const int grid = (n + 255) / 256;
  if (a.X) k_column_put<<<grid, 256, 0, s>>>(n, X, a.X + col, a.ldx);
  if (a.B) k_column_put<<<grid, 256, 0, s>>>(n, g->ws->b64, a.B + col, a.ldx);
  if (a.R) k_column_put<<<grid, 256, 0, s>>>(n, g->ws->r64, a.R + col, a.ldx);
  NVD_HIP(hipGetLastError());
  nvd_pair_info got;
  NVD_HIP(hipMemcpyAsync(&got, g->ws->info, sizeof(got), hipMemcpyDeviceToHost, s));
  NVD_HIP(hipStreamSynchronize(s));
  got.iters += info->iters;
  got.refine_steps = info->refine_steps;
  got.flags |= NVD_INFO_FP64_FALLBACK;
  *info = got;
  return NVD_OK;
}

// The k pairs (P[:, j], Q[:, j]) of one graph.
nvd_status solve_column(DevGraph* g, int k, const double* P, const double* Q, int64_t ld,
                        const SolveParams& sp, double* d_out, double* X, int64_t ldx,
                        nvd_pair_info* info, hipStream_t s, double* B, double* R) try {
  const bool mixed = sp.precision == NVD_MIXED;
  NVD_TRY(ensure_column(g, s));
  const ColPlan* cp = g->col;
  const long stride = (long)cp->d.slots * kColBS;
  const long cstride = g->n_comp > 1 ? g->n_comp : 0;
  const int chunk = std::min(k, kColChunk);
  const int vecs = sp.tree ? 8 : 4;
  NVD_TRY(ensure_column_ws(&g->col_ws, (size_t)stride * vecs * chunk, (size_t)cstride * chunk, chunk, &g->bytes));
  ColArgs a{};
  a.vecs = vecs;
  if (sp.tree) NVD_TRY(ensure_column_pre(g, sp.achol, cp->d.perm, cp->d.slots, &a.pre));
  a.g = cp->d;
  a.P = P;
  a.Q = Q;
  a.ld = ld;
  a.rtol2 = sp.rtol * sp.rtol;
  a.irtol2 = sp.inner_rtol * sp.inner_rtol;
  a.stall_ratio2 = kStallRatio2;
  if (const char* e = std::getenv("NVD_REFINE_STALL_RATIO2")) {
    const double v = std::strtod(e, nullptr);
    if (v >= 0.0 && v <= 1.0) a.stall_ratio2 = v;
  }
  a.max_iter = sp.max_iter;
  a.max_refine = sp.max_refine;
  a.out_dsq = sp.out_dsq ? 1 : 0;
  a.call = kColOwn;
  const size_t hb = parts_bytes(cp->d.nv);
  const size_t most = ((size_t)kColLds - hb) / (sizeof(double) * kColBS) * kColBS;
  a.lds_n = (int)std::min<size_t>(stride, most);
  // (the forest's augmentation takes kColAugLds values of it, whatever n)
  const size_t least = sp.tree ? (size_t)kColAugLds : 0;
  const size_t bytes = hb + sizeof(double) * std::max<size_t>(a.lds_n, least);
  a.d_out = d_out;
  a.X = X;
  a.B = B;
  a.R = R;
  a.ldx = ldx;
  a.info = g->col_ws.info;
  a.vec = g->col_ws.vec;
  a.stride = stride;
  a.cmean = g->col_ws.vec + g->col_ws.cap_vec;
  a.cstride = cstride;
  auto launch = [&](bool in_fp64, size_t lds, int cols) -> nvd_status {
    return (sp.tree ? launch_column_pre : launch_column_jacobi)(a, !in_fp64, !g->weighted, g->n, cols, lds, s);
  };
  for (int c0 = 0; c0 < k; c0 += chunk) {
    const int cols = std::min(chunk, k - c0);
    a.col0 = c0;
    a.resume = 0;
    NVD_TRY(launch(!mixed, bytes, cols));
    NVD_HIP(hipStreamSynchronize(s));
    const nvd_pair_info* got = g->col_ws.info;
    auto left = [&](int j) { return got[j].status == kColResume; };
    bool any = false;
    for (int j = 0; j < cols; ++j) any = any || left(j);
    if (any && column_fits(g->n, false)) {
      a.resume = 1;
      NVD_TRY(launch(true, hb + sizeof(double) * std::max<size_t>(stride, least), cols));
      NVD_HIP(hipStreamSynchronize(s));
    }
    std::copy(got, got + cols, info + c0);
    for (int j = 0; any && j < cols; ++j)
      if (left(j)) NVD_TRY(finish_multi_kernel(g, c0 + j, j, P, Q, ld, sp, a, &info[c0 + j], s));
  }
  return NVD_OK;
} catch (const std::bad_alloc&) {   // (the layout's host arrays)
  set_error("column solve: out of host memory");
  return NVD_E_NOMEM;
}

// ---------------------------------------------------------------------------
// batches of small graphs
// ---------------------------------------------------------------------------
// Every (graph, pair) is a block, the longest first.  Taken where every graph
// of the batch fits, by the rule of batch_is_faster.
// Beside a sweep over larger graphs the blocks took from it what they saved
// (62 graphs up to 37,000 nodes, 14 pairs: 18.6 / 18.0): such batches are
// swept whole.  Beyond 24 slots a block's iteration takes longer than the
// sweep's (n = 32,000, weighted: 32 us / 26).
constexpr int kColBatchNodes = 24 * kColBS;
// Scratch of one launch at most: far fewer pairs are in flight (two a CU) than
// a batch may have (10^5 graphs of 64 pairs: 210 GB for all at once), and the
// next launch uses the same vectors.  1,365 pairs of the largest graphs.
constexpr size_t kColBatchScratch = (size_t)1 << 30;

// Jobs of one launch.
struct ColChunk {
  int first, count, weighted;
  int slots, nv;                   // the most of its graphs
};

struct ColBatch {
  // the graphs' layouts: their counts, and their arrays in host memory until a
  // call is solved by blocks (others hold nothing of them on the device)
  std::vector<ColGraph> h;
  std::vector<unsigned char> host;
  std::vector<size_t> o_src, entries;
  std::vector<int> weighted, nnz, max_deg;
  int most = 0;                    // nodes of the largest
  unsigned char* blob = nullptr;
  double* weights = nullptr;
  ColGraph* dev = nullptr;
  // jobs of the last call, kept while the pair counts stay the same
  std::vector<int> ks;
  std::vector<ColChunk> chunks;
  ColJob* jobs_dev = nullptr;
  size_t cap_jobs = 0, work = 0;
  ColWs ws;
  int64_t bytes = 0;
};

void free_column_batch(ColBatch* c, int64_t* bytes) {
  if (!c) return;
  *bytes -= c->bytes + (int64_t)(sizeof(double) * (c->ws.cap_vec + c->ws.cap_cm));
  void* ptrs[] = {c->blob, c->weights, c->dev, c->jobs_dev};
  for (void* p : ptrs) (void)hipFree(p);
  free_column_ws(&c->ws);
  delete c;
}

static nvd_status lay_out_batch(int G, const DevGraph* const* graphs, ColBatch** out) {
  int most = 0;
  for (int i = 0; i < G; ++i) most = std::max(most, graphs[i]->n_comp == 1 ? graphs[i]->n : INT32_MAX);
  if (most > kColBatchNodes) return NVD_OK;
  std::vector<ColLayout> lay(G);
  const int nt = (int)std::max(1u, std::min(std::min(16u, std::thread::hardware_concurrency()), (unsigned)G));
  std::atomic<int> next{0};
  std::atomic<bool> failed{false};
  auto run = [&]() {
    try {
      for (int i = next++; i < G && !failed; i = next++) layout_column(graphs[i], &lay[i]);
    } catch (const std::bad_alloc&) {
      failed = true;
    }
  };
  std::vector<std::thread> th;
  try {
    for (int t = 1; t < nt; ++t) th.emplace_back(run);
  } catch (const std::exception&) {}   // (fewer threads, then)
  run();
  for (auto& x : th) x.join();
  if (failed) return NVD_E_NOMEM;
  Blob bl;
  std::unique_ptr<ColBatch> c(new ColBatch());
  c->most = most;
  for (int i = 0; i < G; ++i) {
    const DevGraph* g = graphs[i];
    lay[i].put(&bl);
    c->h.push_back(lay[i].d);
    c->o_src.push_back(lay[i].o_src);
    c->entries.push_back(lay[i].src.size());
    c->weighted.push_back(g->weighted ? 1 : 0);
    c->nnz.push_back(g->nnz);
    c->max_deg.push_back(g->max_deg);
    lay[i] = ColLayout();
  }
  c->host = std::move(bl.h);
  *out = c.release();
  return NVD_OK;
}

// The layouts on the device, with the weights of the batch's graphs.
static nvd_status upload_batch(ColBatch* c, const ColBatchArrays& b, int64_t* bytes, hipStream_t s) {
  if (c->dev) return NVD_OK;
  const size_t G = c->h.size();
  auto doubles = [&](size_t i) {
    return weight_doubles(c->weighted[i] ? c->entries[i] : 0, c->h[i].slots * kColBS);
  };
  size_t nw = 0;
  for (size_t i = 0; i < G; ++i) nw += doubles(i);
  ColGraph* dev = nullptr;
  nvd_status st = NVD_OK;
  hipError_t e = device_alloc((void**)&c->blob, c->host.size());
  if (e == hipSuccess) e = device_alloc((void**)&c->weights, sizeof(double) * nw);
  if (e == hipSuccess) e = device_alloc((void**)&dev, sizeof(ColGraph) * G);
  if (e == hipSuccess) e = hipMemcpyAsync(c->blob, c->host.data(), c->host.size(), hipMemcpyHostToDevice, s);
  std::vector<ColGraph> placed;
  size_t at = 0;
  for (size_t i = 0; e == hipSuccess && st == NVD_OK && i < G; ++i) {
    ColGraph d = place(c->h[i], c->blob);
    st = put_weights(c->weighted[i] ? b.w64 + b.nnz_off[i] : nullptr, b.invd64 + b.node_off[i],
                     b.invd32 + b.node_off[i], &d, c->entries[i],
                     reinterpret_cast<const int*>(c->blob + c->o_src[i]), c->weights + at, s);
    at += doubles(i);
    placed.push_back(d);
  }
  if (e == hipSuccess && st == NVD_OK)
    e = hipMemcpyAsync(dev, placed.data(), sizeof(ColGraph) * G, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess && st == NVD_OK) {
    set_error(std::string("batch layouts: ") + hipGetErrorString(e));
    st = e == hipErrorOutOfMemory ? NVD_E_NOMEM : NVD_E_DEVICE;
  }
  if (st != NVD_OK) {
    for (void* p : {(void*)c->blob, (void*)c->weights, (void*)dev}) (void)hipFree(p);
    c->blob = nullptr;
    c->weights = nullptr;
    return st;
  }
  c->dev = dev;
  const int64_t held = (int64_t)(c->host.size() + sizeof(double) * nw + sizeof(ColGraph) * G);
  c->bytes += held;
  *bytes += held;
  std::vector<unsigned char>().swap(c->host);
  return NVD_OK;
}

ColBatch* make_column_batch(int G, const DevGraph* const* graphs) {
  ColBatch* c = nullptr;
  try {
    if (lay_out_batch(G, graphs, &c) != NVD_OK) return nullptr;
  } catch (const std::bad_alloc&) {
    return nullptr;                // (out of host memory: the batch is swept)
  }
  return c;
}

// Blocks or the sweep: the smaller of an iteration's estimates (us), of blocks the
// longest pair's or what all pairs take on 256 CUs, of the sweep its launches and
// its gathers over all graphs, and again over the largest, which one XCD has.
// Blocks win nearly everywhere (392 batches of 2 to 64 graphs up to 24,000 nodes
// of degree 4 to 120, 1 to 64 pairs: 0.03 to 0.8 of the sweep's time; ms a call,
// block / sweep: 47 graphs up to 9,900 nodes, 5 pairs 1.2 / 6.4; 64 up to 17,000,
// 16 pairs 4.5 / 13.0), also on dense graphs whose rows the sweep cuts into
// segments (n = 20,000 of degree 200, one pair 20 / 43).  They lose with few pairs
// on a few graphs whose entries leave the L2 in rows that the sweep does not cut
// (2 of n = 16,000, degree 120, 4 pairs: 8.6 / 3.3).  Both estimates are off by half
// at times, so blocks are left only where they look slower by as much.
static bool batch_is_faster(const ColBatch* c, const std::vector<int>& ks, bool fp64) {
  double longest = 0.0, all = 0.0, entries = 0.0, cut = 0.0;
  int kmax = 1;
  size_t big = 0;
  for (size_t g = 0; g < c->h.size(); ++g) {
    const double t = block_iteration(c->h[g].n, c->nnz[g], c->max_deg[g], c->weighted[g] != 0, fp64);
    if (t > longest) {
      longest = t;
      big = g;
    }
    all += t * ks[g];
    entries += c->nnz[g];
    kmax = std::max(kmax, ks[g]);
    if ((double)c->nnz[g] > (double)kLongRow * c->h[g].n) cut = std::max(cut, (double)c->h[g].n);
  }
  if (stream_bytes(c->nnz[big], c->weighted[big] != 0, fp64) <= 3.5e6) return true;
  int T = 1;
  while (T < kmax) T *= 2;
  const double es = fp64 ? 8.0 : 4.0;
  const double sweep = 22.0 + 1.5 * T + (2.0e-7 * entries + 1.0e-6 * c->nnz[big]) * T * es +
                       (cut > 0.0 ? cut * (T < 4 ? 0.066 : 0.095) : 3.7e-5 * c->nnz[big]);
  return std::max(longest, all / 256.0) <= (cut > 0.0 ? 1.3 : 1.6) * sweep;
}

bool use_column_batch(const ColBatch* c, const std::vector<int>& ks, bool mixed) {
  if (!column_fits(c->most, mixed)) return false;
  if (const char* e = std::getenv("NVD_COLUMN")) return e[0] != '0';   // 0 never, 1 wherever it fits
  return batch_is_faster(c, ks, !mixed);
}

nvd_status solve_column_batch(ColBatch* c, const ColBatchArrays& arrays, const std::vector<int>& ks,
                              const nvd_opts& o, const double* P,
                              const double* Q, double* d_out, double* X, nvd_pair_info* info, int64_t* bytes,
                              hipStream_t s) try {
  NVD_TRY(upload_batch(c, arrays, bytes, s));
  const int G = (int)c->h.size();
  int K = 0;
  for (const int k : ks) K += k;
  if (c->ks != ks) {
    // (every call waits for its launches: the jobs may change)
    c->ks.clear();
    std::vector<long> voff(G);
    std::vector<int> out(G), order(G);
    long v = 0;
    int first = 0;
    for (int g = 0; g < G; ++g) {
      voff[g] = v;
      out[g] = first;
      first += ks[g];
      v += (long)c->h[g].n * ks[g];
    }
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return c->h[x].n > c->h[y].n; });
    // unit graphs, then weighted ones (another kernel), in launches whose
    // vectors fit the scratch
    c->work = 0;
    c->chunks.clear();
    std::vector<ColJob> all;
    all.reserve(K);
    for (int w = 0; w < 2; ++w) {
      size_t work = 0;
      bool open = false;
      for (const int g : order) {
        if (c->weighted[g] != w) continue;
        const size_t need = (size_t)4 * c->h[g].slots * kColBS;
        for (int j = 0; j < ks[g]; ++j) {
          if (!open || sizeof(double) * (work + need) > kColBatchScratch) {
            c->chunks.push_back({(int)all.size(), 0, w, 0, 0});
            work = 0;
            open = true;
          }
          ColJob job{};
          job.graph = g;
          job.out = out[g] + j;
          job.voff = job.xoff = voff[g] + j;
          job.ld = job.ldx = ks[g];
          job.work = (long)work;
          all.push_back(job);
          work += need;
          c->work = std::max(c->work, work);
          ColChunk& ch = c->chunks.back();
          ch.count += 1;
          ch.slots = std::max(ch.slots, c->h[g].slots);
          ch.nv = std::max(ch.nv, c->h[g].nv);
        }
      }
    }
    if (c->cap_jobs < all.size()) {
      (void)hipFree(c->jobs_dev);
      c->jobs_dev = nullptr;
      c->bytes -= (int64_t)(sizeof(ColJob) * c->cap_jobs);
      *bytes -= (int64_t)(sizeof(ColJob) * c->cap_jobs);
      c->cap_jobs = 0;
      NVD_HIP(device_alloc((void**)&c->jobs_dev, sizeof(ColJob) * all.size()));
      c->cap_jobs = all.size();
      c->bytes += (int64_t)(sizeof(ColJob) * c->cap_jobs);
      *bytes += (int64_t)(sizeof(ColJob) * c->cap_jobs);
    }
    NVD_HIP(hipMemcpy(c->jobs_dev, all.data(), sizeof(ColJob) * all.size(), hipMemcpyHostToDevice));
    c->ks = ks;
  }
  NVD_TRY(ensure_column_ws(&c->ws, c->work, 0, K, bytes));
  ColArgs a{};
  a.graphs = c->dev;
  a.vecs = 4;
  a.P = P;
  a.Q = Q;
  a.rtol2 = o.rtol * o.rtol;
  a.irtol2 = o.inner_rtol * o.inner_rtol;
  a.stall_ratio2 = kStallRatio2;
  a.max_iter = o.max_iter;
  a.max_refine = o.max_refine;
  a.out_dsq = 0;
  a.call = o.precision != NVD_MIXED && o.max_refine < 3 ? kColBatchTwo : kColBatch;
  a.d_out = d_out;
  a.X = X;
  a.info = c->ws.info;
  a.vec = c->ws.vec;
  for (const ColChunk& ch : c->chunks) {
    const size_t fit = ((size_t)kColLds - parts_bytes(ch.nv)) / (sizeof(double) * kColBS);
    a.lds_n = (int)std::min<size_t>(ch.slots, fit) * kColBS;
    a.jobs = c->jobs_dev + ch.first;
    NVD_TRY(launch_column_jacobi(a, o.precision == NVD_MIXED, ch.weighted == 0, ch.slots * kColBS, ch.count,
                                 parts_bytes(ch.nv) + sizeof(double) * (size_t)a.lds_n, s));
  }
  NVD_HIP(hipStreamSynchronize(s));
  std::copy(c->ws.info, c->ws.info + K, info);
  return NVD_OK;
} catch (const std::bad_alloc&) {
  set_error("batch solve: out of host memory");
  return NVD_E_NOMEM;
}

}  // namespace nvd
