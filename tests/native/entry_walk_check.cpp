// CPU check of csrc/entry_walk.hpp: on the largest graphs (up to 2^31 - 2
// entries) and the smallest, every thread's entries lie within the graph, rise
// by the grid's step and end, and the threads together take each entry once.
#include <climits>
#include <cstdio>
#include <vector>

#include "entry_walk.hpp"

int main() {
  int bad = 0;
  auto fail = [&](const char* what, long count, long blocks, long thread) {
    std::printf("FAIL %s: count %ld blocks %ld thread %ld\n", what, count, blocks, thread);
    ++bad;
  };
  // one thread's entries: in range, one step apart, and as many as there are
  auto thread_ok = [&](int count, unsigned blocks, unsigned block, unsigned t) {
    const long first = (long)block * nvd::kEntryBS + t, step = (long)blocks * nvd::kEntryBS;
    const long want = first < count ? (count - first + step - 1) / step : 0;
    long seen = 0;
    bool ok = true;
    struct Stop {};
    try {
      nvd::for_entries(block, blocks, t, count, [&](int e) {
        ok = ok && e >= 0 && e < count && e == first + seen * step;
        if (!ok || ++seen > want) throw Stop();
      });
    } catch (Stop) {
      ok = false;
    }
    if (!ok || seen != want) fail("a thread's entries", count, blocks, first);
  };
  for (int count : {INT_MAX - 1, INT_MAX - (1 << 19), INT_MAX - (1 << 24), INT_MAX - 2 * (1 << 24), (1 << 24) + 1})
    for (unsigned blocks : {(unsigned)nvd::entry_grid(count), 2048u})
      for (unsigned block : {0u, 1u, blocks / 2, blocks - 2, blocks - 1})
        for (unsigned t : {0u, 1u, 255u}) thread_ok(count, blocks, block, t);
  // together: each entry once
  for (int count : {0, 1, 255, 256, 257, 1000, 70000}) {
    for (unsigned blocks : {1u, 3u, (unsigned)nvd::entry_grid(count)}) {
      std::vector<int> hits(count + 1, 0);
      for (unsigned b = 0; b < blocks; ++b)
        for (unsigned t = 0; t < (unsigned)nvd::kEntryBS; ++t)
          nvd::for_entries(b, blocks, t, count, [&](int e) { ++hits[e]; });
      for (int e = 0; e < count; ++e)
        if (hits[e] != 1) {
          fail("entry not taken once", count, blocks, e);
          break;
        }
    }
  }
  if (nvd::entry_grid(0) != 1 || nvd::entry_grid((long)INT_MAX - 1) != nvd::kEntryBlocks) fail("grid", 0, 0, 0);
  if (!bad) std::printf("ok\n");
  return bad ? 1 : 0;
}
