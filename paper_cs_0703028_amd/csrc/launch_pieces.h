// Launches over groups of cells within what one launch may hold.  Host code
// without HIP (a CPU test compiles it alone).
#pragma once
#include <algorithm>
#include <cstdint>

namespace rt {

// A launch's blocks times its block's threads, along x, must stay below 2^32
// (the width of the dispatch packet's grid size).  With blocks of 256 threads and
// 8 cells x 256 points of a table that is 137 GB of it.
constexpr int64_t kLaunchThreads = (int64_t(1) << 32) - 1;

inline bool launch_fits(int64_t blocks, int64_t threads) {
  return blocks <= kLaunchThreads / threads;
}

// `groups` groups of per_group blocks each, and `extra` blocks behind those of
// the last group, in as few launches as hold them: launch(first group, groups,
// blocks, whether the extra blocks follow) for each, until one fails (returns
// false).  False as well where one group does not fit.
template <class F>
bool for_pieces(int64_t groups, int64_t per_group, int64_t extra, int64_t threads, F launch) {
  if (groups <= 0 || per_group <= 0) return true;
  const int64_t most = (kLaunchThreads / threads - extra) / per_group;
  if (most < 1) return false;
  for (int64_t g = 0; g < groups; g += most) {
    const int64_t n = std::min(most, groups - g);
    if (!launch(g, n, n * per_group, g + n == groups)) return false;
  }
  return true;
}

}  // namespace rt
