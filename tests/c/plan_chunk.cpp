// The chunk length of the entity layouts: shorter than the default only where a
// chunk holds several rows and packing splits few of them, and never with more
// partial slots than the default length without packing.  Exit status 0 when
// every check holds.  Built and run by tests/test_plan_chunk.py.
#define main plan_sanitized_main
#include "plan_sanitized.cpp"
#undef main

static int64_t slots(const LayoutHost &L, int64_t n_e, int32_t chunk, bool pack) {
  PlanOptions po;
  po.chunk = chunk;
  po.n_xcd = 8;
  po.n_ids_a = po.n_ids_b = n_e;
  po.wide = pack ? 1024 : 0;
  po.pack = pack;
  return plan_layout(L, po).n_slots;
}

// want0, want1: the forward and dX layouts' chunk lengths, 0 for the default.
static void chunk_case(const char *what, int64_t n_e, const std::vector<int32_t> &s,
                       const std::vector<int32_t> &o, int32_t want0, int32_t want1) {
  const int64_t n_t = (int64_t)s.size();
  std::mt19937_64 g(5);
  std::vector<int32_t> r(n_t);
  for (auto &x : r) x = (int32_t)(g() % 50);
  LayoutHost L[3];
  build_layouts(n_e, 50, n_t, s.data(), r.data(), o.data(), nullptr, false, false, L);
  for (int k = 0; k < 2; ++k) {
    const int32_t base = default_chunk(n_t + n_e), c = entity_chunk(L[k], n_e);
    const int32_t want = k ? want1 : want0;
    CHECK(c == (want ? want : base), "%s, layout %d: chunks of %d, default %d", what, k, c, base);
    const int64_t now = slots(L[k], n_e, c, true), before = slots(L[k], n_e, base, false);
    CHECK(now <= before, "%s, layout %d: %lld slots, %lld before", what, k, (long long)now,
          (long long)before);
    std::printf("%s, layout %d: default %d, chunk %d, slots %lld (%lld)\n", what, k, base, c,
                (long long)now, (long long)before);
  }
}

// Objects with exactly `per` triples each about entities at random.
static void rows_case(const char *what, int64_t n_e, int64_t per, int32_t want0, int32_t want1) {
  std::mt19937_64 g(17);
  std::vector<int32_t> s, o;
  for (int64_t q = 0; q < n_e; ++q)
    for (int64_t i = 0; i < per; ++i) {
      s.push_back((int32_t)(g() % n_e));
      o.push_back((int32_t)q);
    }
  chunk_case(what, n_e, s, o, want0, want1);
}

int main() {
  // 2.4 M entries (the grid of 700 x 700 cells) default to 64, 450 k to 16.
  for (int64_t n : {300, 700}) {  // a grid of n x n cells and their four neighbours
    std::vector<int32_t> s, o;
    for (int64_t i = 0; i < n; ++i)
      for (int64_t j = 0; j < n; ++j)
        for (int d = 0; d < 4; ++d) {
          const int64_t a = i + (d == 0) - (d == 1), b = j + (d == 2) - (d == 3);
          if (a < 0 || b < 0 || a >= n || b >= n) continue;
          s.push_back((int32_t)(i * n + j));
          o.push_back((int32_t)(a * n + b));
        }
    chunk_case(n == 300 ? "grid 300" : "grid 700", n * n, s, o, n == 300 ? 0 : 32,
               n == 300 ? 0 : 32);
  }
  rows_case("10 a row", 200'000, 10, 0, 0);  // 2.2 M entries: 64; 32 holds fewer than five rows
  rows_case("6 a row", 500'000, 6, 32, 32);  // 3.5 M: 64
  rows_case("80 a row", 30'000, 80, 0, 0);
  // 8.8 M entries (256): rows of exactly 10 leave 7 of 128 entries and 9 of 64.
  rows_case("10 a row, many", 800'000, 10, 128, 64);
  rows_case("30 a row", 285'000, 30, 0, 0);
  // Two triples in three in rows of 200, few of the rows: their partials count.
  {
    std::mt19937_64 g(3);
    std::vector<int32_t> s, o;
    for (int32_t q = 0; q < 600'000; ++q)
      for (int i = 0; i < (q % 100 == 0 ? 200 : 1); ++i) {
        s.push_back((int32_t)(g() % 600'000));
        o.push_back(q);
      }
    chunk_case("mixed rows", 600'000, s, o, 0, 32);
  }
  // Nothing to sample.
  LayoutHost none;
  none.rows = 9;
  CHECK(entity_chunk(none, 9) == 16, "empty layout");
  if (failures) {
    std::fprintf(stderr, "%d checks failed\n", failures);
    return 1;
  }
  std::printf("chunk lengths hold\n");
  return 0;
}
