// The chunk length of the entity layouts: shorter than the default only where few
// rows would be split, below 128 only where the gathered ids are local too, and
// never with more partial slots than the default length without packing.  Exit status 0 when
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

// `want`: the forward layout's chunk length, 0 for the default.
static void chunk_case(const char *what, int64_t n_e, const std::vector<int32_t> &s,
                       const std::vector<int32_t> &o, int32_t want) {
  const int64_t n_t = (int64_t)s.size();
  std::mt19937_64 g(5);
  std::vector<int32_t> r(n_t);
  for (auto &x : r) x = (int32_t)(g() % 50);
  LayoutHost L[3];
  build_layouts(n_e, 50, n_t, s.data(), r.data(), o.data(), nullptr, false, false, L);
  for (int k = 0; k < 2; ++k) {
    const int32_t base = default_chunk(n_t + n_e), c = entity_chunk(L[k], n_e);
    CHECK(c == (want ? want : base), "%s, layout %d: chunks of %d, default %d", what, k, c, base);
    const int64_t now = slots(L[k], n_e, c, true), before = slots(L[k], n_e, base, false);
    CHECK(now <= before, "%s, layout %d: %lld slots, %lld before", what, k, (long long)now,
          (long long)before);
    std::printf("%s, layout %d: default %d, chunk %d, slots %lld (%lld)\n", what, k, base, c,
                (long long)now, (long long)before);
  }
}

// Rows of `per` triples about entities at random, or within `reach` of the row.
static void rows_case(const char *what, int64_t n_e, int64_t per, int64_t reach, int32_t want) {
  std::mt19937_64 g(17);
  std::vector<int32_t> s, o;
  for (int64_t q = 0; q < n_e; ++q)
    for (int64_t i = 0; i < per; ++i) {
      const int64_t id = reach ? q - reach + (int64_t)(g() % (2 * reach + 1)) : (int64_t)(g() % n_e);
      s.push_back((int32_t)std::min(n_e - 1, std::max<int64_t>(0, id)));
      o.push_back((int32_t)q);
    }
  chunk_case(what, n_e, s, o, want);
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
    chunk_case(n == 300 ? "grid 300" : "grid 700", n * n, s, o, n == 300 ? 0 : 32);
  }
  rows_case("even ids, 10 a row", 200'000, 10, 0, 0);
  rows_case("even ids, 80 a row", 30'000, 80, 0, 0);
  // Above 8.4 M entries (256): halved for rows of up to 16 triples.
  rows_case("even ids, 10 a row, many", 800'000, 10, 0, 128);
  rows_case("even ids, 20 a row", 420'000, 20, 0, 0);
  rows_case("local ids, 4 a row", 400'000, 4, 500, 32);
  rows_case("local ids, 5 a row", 400'000, 5, 500, 0);  // longer than an eighth of 32
  rows_case("local ids, 80 a row", 30'000, 80, 500, 0);
  // One id gathered by nearly every row: alike, not local.
  {
    std::mt19937_64 g(3);
    std::vector<int32_t> s, o;
    for (int32_t q = 0; q < 400'000; ++q)
      for (int i = 0; i < 5; ++i) {
        s.push_back(g() % 10 ? 7 : (int32_t)(g() % 400'000));
        o.push_back(q);
      }
    LayoutHost L[3];
    std::vector<int32_t> r(s.size(), 0);
    build_layouts(400'000, 1, (int64_t)s.size(), s.data(), r.data(), o.data(), nullptr, false,
                  false, L);
    CHECK(!local_ids(L[0]), "one hot id");
  }
  // Nothing to sample.
  LayoutHost none;
  none.rows = 9;
  CHECK(!local_ids(none) && entity_chunk(none, 9) == 16, "empty layout");
  if (failures) {
    std::fprintf(stderr, "%d checks failed\n", failures);
    return 1;
  }
  std::printf("chunk lengths hold\n");
  return 0;
}
