// The int8 product plans of csrc/modular.h as flat integers, for tests/test_modular_plan.py
// (compiled there and linked against the built library; host code only).
#include <cstdint>

#include "modular.h"

namespace {
struct Out {
  int64_t* o;
  int64_t cap, n = 0;
  void put(int64_t v) {
    if (n < cap) o[n] = v;
    ++n;
  }
};
}  // namespace

// -1: no plan; else the count of values: blocks of A, of B, jobs, groups, then the entries.
extern "C" int64_t probe_plan(int64_t m, int64_t n, int64_t k, int S, int T, int w, int64_t* o, int64_t cap) {
  const auto pl = mdg::modular_plan(m, n, k, S, T, w);
  if (!pl) return -1;
  Out out{o, cap};
  for (int64_t v : {static_cast<int64_t>(pl->a.size()), static_cast<int64_t>(pl->b.size()),
                    static_cast<int64_t>(pl->jobs.size()), static_cast<int64_t>(pl->groups.size()),
                    static_cast<int64_t>(pl->pa), static_cast<int64_t>(pl->pb), static_cast<int64_t>(pl->planes),
                    static_cast<int64_t>(mdg::modular_accum_fits(*pl, w))})
    out.put(v);
  for (const auto* v : {&pl->a, &pl->b})
    for (const mdg::ModBlock& b : *v)
      for (int64_t x : {b.lo + 0, b.bits + 0, b.count + 0, b.residue + 0, b.scaled + 0}) out.put(x);
  for (const mdg::ModJob& j : pl->jobs)
    for (int64_t x : {j.a + 0, j.b + 0, j.da + 0, j.db + 0, j.nseg + 0, j.mod + 0, j.out + 0}) out.put(x);
  for (const mdg::ModGroup& g : pl->groups)
    for (int64_t x : {g.shift + 0, g.out + 0, g.residue + 0, g.count + 0}) out.put(x);
  return out.n;
}

extern "C" int probe_modulus(int i) { return mdg::kModuli[i]; }
extern "C" int probe_level_passes_exact(int pairs, int64_t k, int w) { return mdg::level_passes_exact(pairs, k, w); }
extern "C" int probe_split_fits(int64_t m, int64_t n, int64_t k) { return mdg::modular_split_fits(m, n, k); }
