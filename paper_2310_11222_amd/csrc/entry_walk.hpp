// How the threads of a grid share `count` CSR entries (plain C++, so that the
// same code is compiled into the kernels and into a CPU test).
//
// A graph may hold up to 2^31 - 2 entries: the index of the last step, which
// ends the loop, lies past what an int holds, so it is counted in 64 bits.
#pragma once

#ifndef NVD_HD
#if defined(__HIPCC__)
#define NVD_HD __host__ __device__
#else
#define NVD_HD
#endif
#endif

namespace nvd {

constexpr int kEntryBS = 256;        // threads per block
constexpr long kEntryBlocks = 65536; // blocks at most

// f(e) on the entries of thread `thread` of block `block`.
template <class F>
NVD_HD inline void for_entries(unsigned block, unsigned blocks, unsigned thread, int count, F&& f) {
  const long step = (long)blocks * kEntryBS;
  for (long e = (long)block * kEntryBS + thread; e < count; e += step) f((int)e);
}

// Blocks for `work` threads.
inline int entry_grid(long work) {
  const long blocks = (work + kEntryBS - 1) / kEntryBS;
  return (int)(blocks < 1 ? 1 : (blocks > kEntryBlocks ? kEntryBlocks : blocks));
}

}  // namespace nvd
