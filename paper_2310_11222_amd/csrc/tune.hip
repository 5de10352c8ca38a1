// Autotuner for the tile: the number of right-hand-side columns per solve
// pass (T) and the neighbour lanes per row of the Laplacian apply (NL).
//
// Wider tiles read the CSR fewer times and gather longer rows of X per
// neighbour (fewer, fuller memory transactions); narrower tiles keep the
// solver's vectors small enough to stay in the last-level cache, which the
// vector passes of every iteration (update, direction) feel as much as the
// apply.  Which wins depends on the graph, so the candidates are timed on the
// graph itself: for each T the apply alone picks NL, then one whole CG
// iteration (apply, update, direction) with that NL is timed, and the T
// minimising the time for all k columns (full tiles and the rest) is cached in
// the graph handle per (precision, k bucket).
#include <algorithm>
#include <cstdlib>

#include "device_common.hpp"

namespace nvd {

static int log2i(int v) {
  int l = 0;
  while ((1 << (l + 1)) <= v) ++l;
  return l;
}

static bool tuning_disabled() {
  const char* e = std::getenv("NVD_TUNE");
  return e && e[0] == '0';
}

// Heuristic used when tuning is off: the largest power of two <= min(k, 32).
static int heuristic_tile(int k) {
  int T = 1;
  while (T * 2 <= k && T * 2 <= 32) T *= 2;
  return T;
}

static nvd_status time_spmm(DevGraph* g, int prec, int T, int nl, hipStream_t s, float* ms) {
  Workspace* ws = g->ws;
  SpmmCall sc{};
  sc.g = g;
  sc.prec = prec;
  sc.T = T;
  sc.nl = nl;
  sc.x = prec == 0 ? (const void*)ws->p64 : (const void*)ws->p32;
  sc.ldx = T;
  sc.y = prec == 0 ? (void*)ws->q64 : (void*)ws->q32;
  sc.ldy = T;
  sc.epi = EPI_PLAIN;
  hipEvent_t a, b;
  NVD_HIP(hipEventCreate(&a));
  NVD_HIP(hipEventCreate(&b));
  nvd_status st = launch_spmm(sc, ws->red, s);   // warm-up
  const int reps = 3;
  if (st == NVD_OK) st = hipEventRecord(a, s) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
  for (int i = 0; i < reps && st == NVD_OK; ++i) st = launch_spmm(sc, ws->red, s);
  if (st == NVD_OK) st = hipEventRecord(b, s) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
  if (st == NVD_OK) st = hipEventSynchronize(b) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
  float t = 0.0f;
  if (st == NVD_OK) st = hipEventElapsedTime(&t, a, b) == hipSuccess ? NVD_OK : NVD_E_DEVICE;
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  *ms = t / reps;
  if (st != NVD_OK) set_error("autotuner: timing failed");
  return st;
}

int tuned_nl(const DevGraph* g, int precision, int T) {
  const int p = precision == NVD_MIXED ? 1 : 0;
  const int nl = g->tuned_nl[p][log2i(T)];
  return nl > 0 ? nl : default_nl(T);
}

int untimed_tile(const DevGraph* g, int k, int precision) {
  if (k <= 8 || g->n < 4096) return heuristic_tile(k);
  const int p = precision == NVD_MIXED ? 1 : 0;
  const int t = g->tuned_tile[p][std::min(log2i(k), 7)];
  return t > 0 ? t : heuristic_tile(k);
}

// Estimated time (us) of one CG iteration of a tile, for the choice between
// covers of a ragged rest only: launch and reduction latency, one line
// request per gather up to 64 bytes of row (a wider row costs by its size),
// and ten vector passes at streaming rate.  On the 10^7-node power-law graph
// (FP32) it gives 2.7 ms at T = 16 (measured 2.4) and 1.6 at T = 1 (row-wise
// 1.3); at 10^5 nodes 18 + 23 + 14 us at T = 32.
static double iteration_estimate(const DevGraph* g, int T, const SolveParams& sp) {
  const double es = sp.precision == NVD_MIXED ? 4.0 : 8.0;
  const double row = T * es;
  const double n = g->n;
  if (g->n_comp == 1 && !sp.tree && !sp.warm && n * T <= 262144.0) return 22.0 + 8.0e-5 * n * T;   // one launch
  // (an explicit preconditioner's solve costs some twenty passes in FP64)
  const double passes = sp.tree ? 10.0 + 160.0 / es : 10.0;
  // several components: their means are taken by a block each, around every
  // inner solve, and the largest one's time, most of a tile's where it is a giant
  // one, grows with the columns (ER n = 3 10^5 of degree 10, 14 components, mixed:
  // 2.8 ms a column; 5 pairs 22.7 ms as a tile of 8, 16.0 as 4 and 1)
  const double means = g->n_comp > 1 ? (sp.precision == NVD_MIXED ? 4.0e-4 : 2.6e-4) * g->max_comp * T : 0.0;
  return (sp.tree ? 60.0 : 18.0) + means + 2.0e-5 * g->nnz * std::max(1.0, row / 84.0) + n * row * passes / 5.5e6;
}

int next_tile(const DevGraph* g, int k, int left, int tile, const SolveParams& sp) {
  // a tile that was picked over wider ones is not exceeded
  const int most = std::max(tile, 2 * tile > k ? std::min({2 * tile, kMaxTile, g->tile_most}) : tile);
  if (left >= 2 * tile || left >= most) return tile;
  int wide = 1;                                  // one tile over all that is left
  while (wide < left && wide < most) wide *= 2;
  if (wide == left) return wide;
  // best[r]: least time for r columns; the tile that it starts with
  double best[kMaxTile + 1];
  int take[kMaxTile + 1];
  best[0] = 0.0;
  for (int r = 1; r <= left; ++r) {
    best[r] = 1e300;
    for (int T = 1; T <= wide; T *= 2) {
      const double t = iteration_estimate(g, T, sp) + best[std::max(0, r - T)];
      if (t < best[r]) {
        best[r] = t;
        take[r] = T;
      }
      if (T >= r) break;                         // one tile holds all r
    }
  }
  return take[left];
}

int narrower_tile(DevGraph* g, int left, int tile, int T) {
  int narrow = tile;
  while (narrow > left) narrow >>= 1;
  if (narrow >= T) return 0;
  g->tile_most = narrow;
  // the workspace that T left is wider than what follows needs
  if (g->ws) {
    g->bytes -= g->ws->bytes;
    free_workspace(g->ws);
    g->ws = nullptr;
  }
  set_error("");
  return narrow;
}

int choose_tile(DevGraph* g, int k, int precision, hipStream_t s) {
  if (k <= 8 || g->n < 4096 || tuning_disabled()) return heuristic_tile(k);
  const int p = precision == NVD_MIXED ? 1 : 0;
  const int kb = std::min(log2i(k), 7);
  if (g->tuned_tile[p][kb] > 0) return g->tuned_tile[p][kb];
  // the SpMM of the inner solver dominates: FP32 for MIXED, FP64 otherwise
  const int prec = p;
  int tmax = 1;
  while (tmax * 2 <= k && tmax * 2 <= kMaxTile) tmax *= 2;
  if (ensure_workspace(g, tmax, prec == 1) != NVD_OK) return heuristic_tile(k);
  double best = 1e30;
  int bestT = heuristic_tile(k);
  for (int T = 8; T <= tmax; T *= 2) {
    float best_apply = 1e30f;
    int nlT = default_nl(T);
    for (int nl = 1; nl <= spmm_max_nl(prec, T); nl *= 2) {
      float ms = 0.0f;
      if (time_spmm(g, prec, T, nl, s, &ms) != NVD_OK) return heuristic_tile(k);
      if (ms < best_apply) {
        best_apply = ms;
        nlT = nl;
      }
    }
    g->tuned_nl[p][log2i(T)] = nlT;
    float it_ms = 0.0f;
    if (time_cg_iteration(g, prec, T, nlT, s, &it_ms) != NVD_OK) return heuristic_tile(k);
    // full tiles, then the rest in the cover that next_tile takes for it
    SolveParams sp{};
    sp.precision = precision;
    double rest = 0.0;
    for (int left = k % T; left > 0;) {
      const int Tr = next_tile(g, k, left, T, sp);
      rest += iteration_estimate(g, Tr, sp) / iteration_estimate(g, T, sp);
      left -= Tr;
    }
    const double total = ((double)(k / T) + rest) * it_ms;
    if (total < best) {
      best = total;
      bestT = T;
    }
  }
  g->tuned_tile[p][kb] = bestT;
  return bestT;
}

}  // namespace nvd

extern "C" nvd_status nvd_tune_query(nvd_graph* h, int32_t k, int32_t precision, int32_t* tile,
                                     int32_t* nl, void* stream) {
  using namespace nvd;
  if (!h || !tile || !nl || k < 1 || (precision != NVD_FP64 && precision != NVD_MIXED)) {
    set_error("nvd_tune_query: bad argument");
    return NVD_E_ARG;
  }
  DevGraph* g = h->g;
  *tile = choose_tile(g, k, precision, reinterpret_cast<hipStream_t>(stream));
  *nl = tuned_nl(g, precision, *tile);
  return NVD_OK;
}
