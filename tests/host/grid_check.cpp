// Checks of csrc/grid.h: the slices of a launch cover every tile once, in order, each below
// 2^32 threads.  tests/test_host_blocks.py builds and runs this.
#include <cstdio>

#include "grid.h"

int main() {
  int fail = 0;
  auto check = [&](bool ok, const char* what, long long n, long long per) {
    if (!ok) std::fprintf(stderr, "FAIL %s: %lld tiles of %lld threads\n", what, n, per), ++fail;
  };
  const int64_t limit = int64_t{1} << 32;
  for (int64_t per : {int64_t{256}, int64_t{2048}, int64_t{65536}, int64_t{98304}, int64_t{6815744}, limit / 2, limit - 1})
    for (int64_t n : {int64_t{1}, int64_t{2}, (limit - 1) / per, limit / per, limit / per + 1, 3 * (limit / per) + 2}) {
      if (n < 1 || n > (int64_t{1} << 31) - 1) continue;
      int64_t at = 0;
      const int e = spanq::launch_in_slices(n, per, 7, [&](int64_t t0, int64_t nt) {
        check(t0 == at && nt >= 1 && nt * per < limit, "slice", n, per);
        at += nt;
        return 0;
      });
      check(e == 0 && at == n, "cover", n, per);
      if (n * per < limit) {
        int calls = 0;
        spanq::launch_in_slices(n, per, 7, [&](int64_t, int64_t) { return ++calls, 0; });
        check(calls == 1, "one launch where one is enough", n, per);
      }
    }
  int calls = 0;
  check(spanq::launch_in_slices(int64_t{3}, limit, 7, [&](int64_t, int64_t) { return ++calls, 0; }) == 7 && calls == 0,
        "too large a tile", 3, limit);
  check(spanq::launch_in_slices(int64_t{9}, limit / 2, 7, [&](int64_t, int64_t) { return ++calls == 2 ? 5 : 0; }) == 5 &&
            calls == 2,
        "stops at an error", 9, limit / 2);
  if (!fail) std::printf("all checks passed\n");
  return fail ? 1 : 0;
}
