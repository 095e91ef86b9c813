// The planner's packed rows and wide combine tasks under the same checks as the
// other plans (plan_sanitized.cpp): every triple once, every row written once,
// and what packing is for -- few rows that a chunk could hold are split.  Exit
// status 0 when every check holds.  Built and run by tests/test_plan_pack.py.
#define main plan_sanitized_main
#include "plan_sanitized.cpp"
#undef main

static void pack_case(const char *what, int64_t n_e, int64_t n_r, const std::vector<int32_t> &s,
                      const std::vector<int32_t> &r, const std::vector<int32_t> &o, bool weighted,
                      bool few_splits) {
  const int64_t n_t = (int64_t)s.size();
  std::vector<float> w(weighted ? n_t : 0, 0.5f);
  LayoutHost L[3];
  build_layouts(n_e, n_r, n_t, s.data(), r.data(), o.data(), weighted ? w.data() : nullptr, false,
                false, L);
  for (int k = 0; k < 3; ++k)
    for (int32_t chunk : {8, 16, 24, 256})
      for (int xcd : {1, 8})
        for (int32_t wide : {0, 5, 1024}) {
          PlanOptions po;
          po.chunk = chunk;
          po.fan_in = 3;
          po.n_xcd = xcd;
          po.hub_min = 64;
          po.hub_by_a = k != 2;
          po.n_ids_a = po.n_ids_b = n_e;
          po.wide = wide;
          const PlanHost plain = plan_layout(L[k], po);
          po.pack = true;
          PlanHost P = plan_layout(L[k], po);
          // (few_splits: rows of a few triples, so packing has something to place.)
          if (few_splits && chunk >= 16 && k < 2)
            CHECK(P.n_split_rows * 3 < plain.n_split_rows + 3, "%s: %lld rows split, %lld unpacked",
                  what, (long long)P.n_split_rows, (long long)plain.n_split_rows);
          CHECK((int64_t)P.entries.size() <=
                    (int64_t)plain.entries.size() * 9 / 8 + 2 * chunk * xcd,
                "%s: %zu entries, %zu unpacked", what, P.entries.size(), plain.entries.size());
          // The wide tasks as ordinary ones of a larger fan-in.
          CHECK(P.wide.size() == P.levels.size(), "%s: levels", what);
          if (wide == 0)
            for (const auto &lv : P.wide) CHECK(lv.empty(), "%s: wide tasks", what);
          for (size_t l = 0; l < P.levels.size(); ++l) {
            for (const CombineTask &t : P.levels[l]) CHECK(t.n <= P.fan_in, "%s: narrow task", what);
            for (const CombineTask &t : P.wide[l]) CHECK(t.n > P.fan_in, "%s: wide task", what);
            P.levels[l].insert(P.levels[l].end(), P.wide[l].begin(), P.wide[l].end());
          }
          P.fan_in = std::max(P.fan_in, wide);
          check_plan(L[k], P, chunk, what);
          interpret_plan(L[k], P, chunk, what);
        }
}

int main() {
  std::mt19937_64 g(7);
  for (int rep = 0; rep < 3; ++rep) {
    const int64_t n_e = 400 + rep * 900, n_r = 1 + rep * 40, n_t = n_e * 5;
    std::uniform_int_distribution<int32_t> E(0, (int32_t)n_e - 1), R(0, (int32_t)n_r - 1);
    std::vector<int32_t> s(n_t), r(n_t), o(n_t);
    for (int64_t l = 0; l < n_t; ++l) {
      s[l] = E(g);
      r[l] = R(g);
      o[l] = E(g);
    }
    pack_case("uniform", n_e, n_r, s, r, o, rep == 1, true);
    for (int64_t l = 0; l < n_t; l += 3) s[l] = 3, o[l] = (int32_t)(l % 2);
    pack_case("hubs", n_e, n_r, s, r, o, rep == 2, false);
  }
  pack_case("empty", 9, 2, {}, {}, {}, false, false);
  pack_case("one triple", 9, 2, {4}, {1}, {8}, true, false);
  if (failures) {
    std::fprintf(stderr, "%d checks failed\n", failures);
    return 1;
  }
  std::printf("packed plans hold\n");
  return 0;
}
