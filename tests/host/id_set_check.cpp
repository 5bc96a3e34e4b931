// Checks of csrc/id_set.h against std::set, at the edges of its levels, and of its lowest() on a
// large set whose only members are its last ids: that must not walk the words before them.
// tests/test_host_blocks.py builds and runs this.
#include <chrono>
#include <cstdio>
#include <random>
#include <set>

#include "id_set.h"

static int g_fail = 0;
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "FAIL line %d: %s\n", __LINE__, #cond);         \
      if (++g_fail > 10) return 1;                                         \
    }                                                                      \
  } while (0)

int main() {
  std::mt19937 rng(7);
  for (int64_t n : {int64_t{1}, int64_t{63}, int64_t{64}, int64_t{65}, int64_t{4096}, int64_t{4097}, int64_t{300000}}) {
    spanq::IdSet s;
    s.resize(n);
    std::set<int64_t> ref;
    for (int step = 0; step < 40000; ++step) {
      const int64_t i = static_cast<int64_t>(rng()) % n;
      CHECK(s.contains(i) == (ref.count(i) == 1));
      if (ref.count(i)) {
        s.erase(i);
        ref.erase(i);
      } else if (step % 3 || ref.empty()) {
        s.insert(i);
        ref.insert(i);
      } else {
        CHECK(s.lowest() == *ref.begin());
        s.erase(s.lowest());
        ref.erase(ref.begin());
      }
      CHECK(s.empty() == ref.empty() && s.size() == static_cast<int64_t>(ref.size()));
      if (!ref.empty()) CHECK(s.lowest() == *ref.begin());
      if (step % 10000 == 9999) {
        s.clear();
        ref.clear();
      }
    }
  }
  const int64_t n = int64_t{1} << 28;
  spanq::IdSet s;
  s.resize(n);
  const auto t0 = std::chrono::steady_clock::now();
  for (int k = 0; k < 200000; ++k) {  // walking 65,536 words each time would take 200 times the limit
    s.insert(n - 1 - k % 100);
    CHECK(s.lowest() == n - 1 - k % 100);
    s.erase(n - 1 - k % 100);
  }
  s.insert(n - 1);
  s.clear();
  CHECK(s.empty() && !s.contains(n - 1));
  const double sec = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  std::printf("200000 lowest ids of a sparse set: %.3f s\n", sec);
  CHECK(sec < 0.5);
  if (g_fail == 0) std::printf("all checks passed\n");
  return g_fail ? 1 : 0;
}
