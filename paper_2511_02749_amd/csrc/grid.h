// Launches over more row tiles than one grid takes.
#pragma once
#include <algorithm>
#include <cstdint>

namespace spanq {

// launch(first, count) over tiles 0 .. n - 1 in as few slices as keep a grid's threads below
// 2^32, which is what a launch takes; stops at the first error.  A tile that is too large by
// itself is `too_large`.
template <typename Error, typename Launch>
Error launch_in_slices(int64_t n, int64_t threads_per_tile, Error too_large, Launch&& launch) {
  const int64_t most = ((int64_t{1} << 32) - 1) / threads_per_tile;
  if (most == 0) return too_large;
  for (int64_t first = 0; first < n; first += most) {
    const Error e = launch(first, std::min(most, n - first));
    if (e != Error{}) return e;
  }
  return Error{};
}

}  // namespace spanq
