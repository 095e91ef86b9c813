// How evenly a plan spreads its chunks over the XCD lists, for KBs whose ids are
// a small part of the id space: clustered at its start, spread over it, with and
// without hot ids.  Prints one line per case; exit status 0 when the longest list
// of every layout is within a tenth of the shortest (or a few chunks), and dR's
// chunks gather from as few blocks of the table as its options ask for.  Built and
// run by tests/test_plan_balance.py.
#define main plan_sanitized_main
#include <algorithm>
#include "plan_sanitized.cpp"
#undef main

static void balance_case(const char *what, int64_t n_e, int64_t used, int64_t n_t, int hot) {
  std::mt19937_64 g(11);
  const int64_t n_r = 50;
  std::uniform_int_distribution<int32_t> E(0, (int32_t)used - 1), R(0, (int32_t)n_r - 1);
  std::vector<int32_t> s(n_t), r(n_t), o(n_t);
  for (int64_t l = 0; l < n_t; ++l) {
    s[l] = E(g), r[l] = R(g), o[l] = E(g);
    // Three triples in ten about one of the hot ids, spread over the used ones.
    if (hot && g() % 10 < 3) s[l] = (int32_t)(g() % hot * (used / hot));
    if (hot && g() % 10 < 3) o[l] = (int32_t)(g() % hot * (used / hot));
  }
  LayoutHost L[3];
  build_layouts(n_e, n_r, n_t, s.data(), r.data(), o.data(), nullptr, false, false, L);
  for (int k = 0; k < 3; ++k)
    for (int class_b = 0; class_b <= (k == 2); ++class_b) {
      PlanOptions po;
      po.chunk = 16;
      po.n_xcd = 8;
      po.hub_by_a = k != 2;
      po.n_ids_a = po.n_ids_b = n_e;
      po.class_by_b = class_b != 0;
      po.a_blocks = k == 2 ? 64 : 0;
      po.wide = 1024;
      po.pack = true;
      PlanHost P = plan_layout(L[k], po);
      // The wide tasks as ordinary ones of a larger fan-in.
      for (size_t l = 0; l < P.levels.size(); ++l)
        P.levels[l].insert(P.levels[l].end(), P.wide[l].begin(), P.wide[l].end());
      P.fan_in = po.wide;
      check_plan(L[k], P, po.chunk, what);
      interpret_plan(L[k], P, po.chunk, what);
      int64_t lo = P.n_chunks, hi = 0;
      std::printf("%s, layout %d, class_b %d:", what, k, class_b);
      for (int x = 0; x < P.n_xcd; ++x) {
        const int64_t n = P.xcd_chunk[x + 1] - P.xcd_chunk[x];
        lo = std::min(lo, n), hi = std::max(hi, n);
        std::printf(" %lld", (long long)n);
      }
      std::printf("\n");
      CHECK(hi <= lo + lo / 10 + 4, "%s, layout %d, class_b %d: lists of %lld to %lld chunks", what,
            k, class_b, (long long)lo, (long long)hi);
    }
}

// dR with classes of the gathered ids: half of the chunks (more than half of the
// triples are not among the heaviest ids, which any list may hold) stay within
// two of the a_blocks blocks of a class's range of the ids.
static void window_case() {
  const int64_t n_e = 400'000, n_r = 10, n_t = 800'000;
  std::mt19937_64 g(23);
  std::vector<int32_t> s(n_t), r(n_t), o(n_t);
  for (int64_t l = 0; l < n_t; ++l)
    s[l] = (int32_t)(g() % n_e), r[l] = (int32_t)(g() % n_r), o[l] = (int32_t)(g() % n_e);
  LayoutHost L[3];
  build_layouts(n_e, n_r, n_t, s.data(), r.data(), o.data(), nullptr, false, false, L);
  for (int32_t blocks : {16, 64}) {
    PlanOptions po;
    po.chunk = 64;
    po.n_xcd = 8;
    po.hub_by_a = false;
    po.n_ids_a = po.n_ids_b = n_e;
    po.a_blocks = blocks;
    po.pack = true;
    const PlanHost P = plan_layout(L[2], po);
    std::vector<int64_t> span;
    for (int64_t c = 0; c < P.n_chunks; ++c) {
      int32_t lo = INT32_MAX, hi = -1;
      for (int64_t p = c * po.chunk; p < (c + 1) * po.chunk; ++p)
        if (P.entries[p].x >= 0) {
          lo = std::min(lo, P.entries[p].x & kIdMask);
          hi = std::max(hi, P.entries[p].x & kIdMask);
        }
      if (hi >= 0) span.push_back(hi - lo);
    }
    std::nth_element(span.begin(), span.begin() + (std::ptrdiff_t)(span.size() / 2), span.end());
    const int64_t median = span[span.size() / 2], most = 2 * n_e / po.n_xcd / blocks;
    std::printf("%d blocks: chunks gather from %lld ids (median)\n", blocks, (long long)median);
    CHECK(median <= most, "%d blocks: chunks over %lld ids, at most %lld", blocks,
          (long long)median, (long long)most);
  }
}

int main() {
  // Above 4 ids per triple and 2^20 more: the id space counts as sparse.
  const int64_t n_e = 4'000'000, n_t = 300'000;
  balance_case("clustered", n_e, n_e / 10, n_t, 0);
  balance_case("clustered, hot ids", n_e, n_e / 10, n_t, 20);
  balance_case("spread", n_e, n_e, n_t, 0);
  balance_case("spread, hot ids", n_e, n_e, n_t, 20);
  // The same ids in a space of their own size: the dense path.
  balance_case("dense", n_e / 10, n_e / 10, n_t, 0);
  balance_case("dense, hot ids", n_e / 10, n_e / 10, n_t, 20);
  window_case();
  if (failures) {
    std::fprintf(stderr, "%d checks failed\n", failures);
    return 1;
  }
  std::printf("lists balanced\n");
  return 0;
}
