// The work lists of the kernels that take any number of query heads per kv head against those of
// the MFMA kernel, over random plans and decode steps: three pools go through the same stream,
// one per tiling, and every caller row has to see the same keys (page, slot, position, shift) in
// each, as the kernel reads them (key lists page by page, or tile records).  Also the generic
// kernel's row tiles: each starts where a page of its span does, or ends with the one it starts
// in.  tests/test_host_blocks.py builds and runs this.
#include <algorithm>
#include <array>
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "planner.h"
#include "spanq.h"

using namespace spanq;

static int g_fail = 0;
#define CHECK(cond, ...)                                                   \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "FAIL line %d (%s): ", __LINE__, #cond);        \
      std::fprintf(stderr, __VA_ARGS__);                                   \
      std::fprintf(stderr, "\n");                                          \
      if (++g_fail > 10) std::exit(1);                                     \
    }                                                                      \
  } while (0)

namespace {

using Key = std::array<int32_t, 4>;  // page, slot, position, shift
using Seen = std::map<int64_t, std::vector<Key>>;  // caller row -> keys it sees, sorted

// What the rows of `tiles` see.  A row's keys may be spread over the parts of its tile; no key
// may come twice.
Seen rows_see(const std::vector<WorkTile>& tiles, const std::vector<KvPage>& kv, const std::vector<TileRec>& kt,
              const Tiling& t, int ps, int max_rows) {
  Seen out;
  for (const WorkTile& w : tiles) {
    CHECK(w.n_rows >= 1 && w.n_rows <= max_rows, "rows of a tile: %d", w.n_rows);
    std::vector<Key> keys;
    if (t.pad4) {
      CHECK(w.kv_begin % 4 == 0 && w.kv_end % 4 == 0, "whole tiles");
      for (int32_t j = w.kv_begin / 4; j < w.kv_end / 4; ++j)
        for (int32_t c = 0; c < kt[j].nk; ++c)
          keys.push_back({kt[j].page_id[c / ps], c % ps, kt[j].pos0 + c, kt[j].delta});
    } else {
      for (int32_t i = w.kv_begin; i < w.kv_end; ++i)
        for (int32_t c = 0; c < kv[i].n_valid; ++c) keys.push_back({kv[i].page_id, c, kv[i].pos0 + c, kv[i].delta});
    }
    for (int32_t r = 0; r < w.n_rows; ++r) {
      auto& mine = out[w.q_row0 + r];
      for (const Key& k : keys)
        if (k[2] <= w.q_pos0 + r) mine.push_back(k);
    }
  }
  for (auto& [row, keys] : out) {
    std::sort(keys.begin(), keys.end(), [](const Key& a, const Key& b) { return a[2] < b[2]; });
    for (size_t i = 0; i < keys.size(); ++i)
      CHECK(keys[i][2] == static_cast<int32_t>(i), "row %lld: key %zu is at position %d", static_cast<long long>(row), i,
            keys[i][2]);
  }
  return out;
}

void run(uint64_t seed, int steps) {
  std::mt19937_64 rng(seed);
  auto pick = [&](uint64_t n) { return rng() % n; };
  const int ps = 16;
  const int64_t num_pages = 60 + static_cast<int64_t>(pick(200));
  std::vector<std::vector<int32_t>> frags, prefixes, crosses;
  auto fill = [&](std::vector<std::vector<int32_t>>& to, std::initializer_list<int> lens, int base) {
    for (int l : lens) {
      to.emplace_back(l);
      for (auto& x : to.back()) x = base + static_cast<int32_t>(pick(50));
    }
  };
  fill(frags, {0, 1, 5, 16, 17, 31, 47, 64, 80, 100, 130}, 0);
  fill(prefixes, {0, 5, 16, 33}, 100);
  fill(crosses, {0, 1, 9, 16, 40, 77}, 1000);
  std::vector<PoolIndex> pools;
  pools.reserve(3);
  for (int i = 0; i < 3; ++i) pools.emplace_back(num_pages, ps, SPAN_HASH_SPAN);
  long plans = 0, decodes = 0, rows_compared = 0;
  for (int s = 0; s < steps; ++s) {
    const int hkv = 1 << pick(4), g = 1 + static_cast<int>(pick(20)), mg = 1 << pick(4);
    Tiling t[3] = {tiling_for(true, 256 / mg, mg * hkv, hkv), tiling_split(128 / g, hkv),
                   tiling_for(false, 64, g * hkv, hkv)};
    const bool materialize = pick(3) == 0;
    for (Tiling& x : t) {
      x.materialize = materialize;
      if (pick(2)) x.min_split_pages = 2;  // many splits
    }
    std::vector<QueryIn> qs(1 + pick(3));
    int64_t row = 0;
    auto span = [&](const std::vector<int32_t>& v) {
      const SpanIn in{v.data(), static_cast<int32_t>(v.size()), row};
      row += in.n;
      return in;
    };
    for (QueryIn& q : qs) {
      q.prefix = span(prefixes[pick(prefixes.size())]);
      for (uint64_t f = pick(5); f-- > 0;) q.frags.push_back(span(frags[pick(frags.size())]));
      q.cross = span(crosses[pick(crosses.size())]);
    }
    Plan P[3];
    int rc[3];
    std::string msg;
    for (int i = 0; i < 3; ++i) rc[i] = pools[i].plan(qs, true, t[i], &P[i], &msg);
    CHECK(rc[0] == rc[1] && rc[0] == rc[2], "one pool refuses what another takes");
    if (rc[0]) continue;
    ++plans;
    {  // lists made again for another tiling are those of a plan made for it
      Plan again = P[1];
      pools[1].rebuild_work(&again, t[2]);
      auto bytes = [](const Plan& p) {
        std::string out;
        auto add = [&](const auto& v) {
          out.append(std::to_string(v.size()));
          if (!v.empty()) out.append(reinterpret_cast<const char*>(v.data()), v.size() * sizeof(v[0]));
        };
        add(p.kv), add(p.kv_tiles), add(p.k3_prefill), add(p.k3_cross), add(p.t_prefill), add(p.t_cross);
        add(p.prefill_chunks), add(p.combine);
        for (const auto* runs : {&p.rows_prefill, &p.rows_cross})
          for (const auto& r : *runs) out += " " + std::to_string(r.row0) + "+" + std::to_string(r.n);
        for (int64_t v : {int64_t{p.n_parts}, int64_t{p.n_cross_few}, int64_t{p.kv_splits}, int64_t{p.max_pos},
                          int64_t{p.bm_cross}, p.prefill_pairs, p.cross_pairs, p.cross_kv_pages})
          out += " " + std::to_string(v);
        return out;
      };
      CHECK(bytes(again) == bytes(P[2]), "rebuilt work lists differ");
    }
    auto compare = [&](auto tiles, auto kv, auto kt, int32_t Tiling::*bm, const char* what) {
      const Seen want = rows_see(tiles(P[0]), kv(P[0]), kt(P[0]), t[0], ps, t[0].*bm);
      for (int i = 1; i < 3; ++i) {
        const Seen got = rows_see(tiles(P[i]), kv(P[i]), kt(P[i]), t[i], ps, t[i].*bm);
        CHECK(got == want, "%s rows of tiling %d see other keys", what, i);
      }
      rows_compared += static_cast<long>(want.size());
    };
    auto kv = [](const Plan& p) -> const auto& { return p.kv; };
    auto kt = [](const Plan& p) -> const auto& { return p.kv_tiles; };
    compare([](const Plan& p) -> const auto& { return p.t_prefill; }, kv, kt, &Tiling::bm_prefill, "prefill");
    compare([](const Plan& p) -> const auto& { return p.t_cross; }, kv, kt, &Tiling::bm_cross, "cross");
    // the generic kernel's tiles against the pages of the span that their rows are in
    std::map<int64_t, int64_t> first_of;  // first row of a span -> one past its last
    for (const SpanPlan& sp : P[2].spans) first_of[sp.row] = std::max(first_of[sp.row], sp.row + sp.n_tok);
    auto aligned = [&](const std::vector<WorkTile>& ts) {
      for (const WorkTile& w : ts) {
        auto it = std::prev(first_of.upper_bound(w.q_row0));
        CHECK(w.q_row0 < it->second, "a tile outside every span");
        const int64_t at = (w.q_row0 - it->first) % ps;
        CHECK(at == 0 || at + w.n_rows <= ps, "a tile starts at slot %d and has %d rows", static_cast<int>(at), w.n_rows);
      }
    };
    aligned(P[2].t_prefill);
    aligned(P[2].t_cross);
    while (pick(3) != 0) {  // a decode step of 0 to 70 tokens a query
      std::vector<int32_t> n(qs.size()), had(qs.size());
      std::vector<int64_t> at(qs.size());
      for (size_t q = 0; q < qs.size(); ++q) {
        n[q] = static_cast<int32_t>(pick(2) ? pick(3) : pick(71));
        had[q] = P[2].spans[P[2].query_spans[q].back()].n_tok;
        at[q] = row;
        row += n[q];
      }
      for (int i = 0; i < 3; ++i) rc[i] = pools[i].decode(&P[i], n, at, t[i], &msg);
      CHECK(rc[0] == rc[1] && rc[0] == rc[2], "one pool refuses a step that another takes");
      if (rc[0]) break;
      ++decodes;
      compare([](const Plan& p) -> const auto& { return p.dec.tiles; }, [](const Plan& p) -> const auto& { return p.dec.kv; },
              [](const Plan& p) -> const auto& { return p.dec.kv_tiles; }, &Tiling::bm_cross, "decode");
      for (const WorkTile& w : P[2].dec.tiles)
        for (size_t q = 0; q < qs.size(); ++q)
          if (w.q_row0 >= at[q] && w.q_row0 < at[q] + n[q]) {
            const int64_t slot = (had[q] + w.q_row0 - at[q]) % ps;
            CHECK(slot == 0 || slot + w.n_rows <= ps, "a decode tile starts at slot %d and has %d rows",
                  static_cast<int>(slot), w.n_rows);
          }
    }
    const bool keep = pick(4) != 0;
    for (int i = 0; i < 3; ++i) keep ? pools[i].commit(&P[i]) : pools[i].release(&P[i]);
  }
  std::printf("seed %llu: %ld plans, %ld decode steps, %ld rows compared\n", static_cast<unsigned long long>(seed), plans,
              decodes, rows_compared);
  CHECK(plans > steps / 2 && decodes > steps / 2, "too few plans or steps");
}

}  // namespace

int main() {
  for (uint64_t seed : {1, 2, 3, 4}) run(seed, 250);
  if (g_fail == 0) std::printf("all checks passed\n");
  return g_fail ? 1 : 0;
}
