// The cover of a product's digit pairs by rectangles (modular.h): which
// rectangles are formed by residues, which pairs directly, and the tables the
// kernels read.  Host only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <tuple>

#include "internal.h"
#include "modular.h"

namespace mdg {
namespace {

// Rates of the estimates, measured on MI355X.
constexpr double kInt8Rate = 2.6e15;   // int8 products, op/s
constexpr double kPlaneRate = 4.5e12;  // bytes/s of panels and planes
// seconds per output element of one job besides its products: the tile's first
// loads and its epilogue (about 4 us per 256 x 256 tile on one of 256 CUs), the
// plane written and read, and the residue's part of the accumulation
constexpr double kTileJob = 4e-6 / 256 / 65536;
constexpr double kResidueJob = kTileJob + 2.0 / kPlaneRate + 0.3e-12;
constexpr double kDirectJobCost = kTileJob + 8.0 / kPlaneRate;
constexpr double kPanelByte = 0.3e-12;  // seconds per panel byte of an operand (residue arithmetic and store)

double log2_moduli(int count) {
  double s = 0.0;
  for (int i = 0; i < count; ++i) s += std::log2(static_cast<double>(kModuli[i]));
  return s;
}

// Moduli for |V| < terms 2^bits: M > 2 |V| (with a little room for the rounding
// of sum y_i / m_i); 0 when the moduli do not suffice.
int moduli_for(int bits, double terms) {
  static const std::vector<double> cum = [] {
    std::vector<double> c;
    for (int i = 0; i <= kMaxModuli; ++i) c.push_back(log2_moduli(i));
    return c;
  }();
  const double need = bits + std::log2(terms) + 1.01;
  for (int i = 1; i <= kMaxModuli; ++i)
    if (cum[i] >= need) return i;
  return 0;
}

struct Rect {
  int p, q, u, v;
};

struct Cover {
  double cost = 0.0;
  int u = 0, v = 0;  // first rectangle at the corner; the rest of its rows, then the rest of the columns
};

// Minimum-cost covers of the pairs p < sa, q < sb, p + q <= t by rectangles cut
// off at the corner (0, 0): the largest one of u rows, or single pairs.
class Coverer {
 public:
  Coverer(int S, int w, double k, double product, double panel, int types)
      : n_(S + 1), memo_(static_cast<size_t>(n_) * n_ * 2 * n_), rect_(static_cast<size_t>(n_) * n_, 1e9) {
    for (int u = 1; u <= S; ++u)
      for (int v = 1; v <= S; ++v) {
        double& c = rect_[static_cast<size_t>(u) * n_ + v];
        if (u == 1 && v == 1) {  // its planes are shared with the level's other pairs (about three)
          c = types * (product + 0.35 * kDirectJobCost + 0.5 * panel);
        } else if (w * std::max(u, v) <= kModMaxBits) {
          const int nm = moduli_for(w * (u + v), 2.0 * k);
          if (nm) c = nm * (product + kResidueJob + panel);
        }
      }
  }

  void rects(int sa, int sb, int t, int p0, int q0, std::vector<Rect>* out) {
    if (t < 0 || sa <= 0 || sb <= 0) return;
    sa = std::min(sa, t + 1);
    sb = std::min(sb, t + 1);
    const Cover c = at(sa, sb, t);
    out->push_back(Rect{p0, q0, c.u, c.v});
    rects(sa - c.u, c.v, t - c.u, p0 + c.u, q0, out);
    rects(sa, sb - c.v, t - c.v, p0, q0 + c.v, out);
  }

 private:
  double cost(int sa, int sb, int t) {
    if (t < 0 || sa <= 0 || sb <= 0) return 0.0;
    return at(std::min(sa, t + 1), std::min(sb, t + 1), t).cost;
  }
  Cover at(int sa, int sb, int t) {
    Cover& slot = memo_[(static_cast<size_t>(t) * n_ + sa) * n_ + sb];
    if (slot.u) return slot;
    Cover best;
    best.cost = 1e18;
    for (int u = 1; u <= sa; ++u) {
      const int vmax = std::min(sb, t - u + 2);
      for (int pass = 0; pass < 2; ++pass) {
        const int v = pass ? 1 : vmax;
        if (v < 1 || (pass && (vmax == 1 || u > 1))) continue;
        // rectangles of several pairs reach the cutoff (their weight is then 1)
        if (u + v > 2 && u + v - 2 != t) continue;
        const double c = rect_[static_cast<size_t>(u) * n_ + v] + cost(sa - u, v, t - u) + cost(sa, sb - v, t - v);
        if (c < best.cost) best = Cover{c, u, v};
      }
    }
    return memo_[(static_cast<size_t>(t) * n_ + sa) * n_ + sb] = best;
  }

  int n_;
  std::vector<Cover> memo_;
  std::vector<double> rect_;
};

// The tables for one cover, at most `longest` rectangles per job; false when a limit
// of the kernels does not hold.
bool build(const std::vector<Rect>& rects, int64_t longest, int64_t k, int S, int T, int w, ModPlan* pl) {
  const int c = sub_digits(w), types = c * (c + 1) / 2;
  // rectangles grouped by (direct or bits, p1 + q1), in order of p0
  std::map<std::tuple<int, int>, std::vector<Rect>> by;
  for (const Rect& r : rects) {
    const bool direct = r.u == 1 && r.v == 1;
    by[std::make_tuple(direct ? 0 : r.u + r.v, r.p + r.u - 1 + r.q + r.v - 1)].push_back(r);
  }
  // direct digits: A's ascending, B's descending, so that the pairs of a level run
  // along both
  std::vector<int> da, db;
  for (const Rect& r : rects)
    if (r.u == 1 && r.v == 1) {
      da.push_back(r.p);
      db.push_back(r.q);
    }
  auto uniq = [](std::vector<int>* v) {
    std::sort(v->begin(), v->end());
    v->erase(std::unique(v->begin(), v->end()), v->end());
  };
  uniq(&da);
  uniq(&db);
  std::reverse(db.begin(), db.end());
  auto lo_of = [&](int p0, int u) { return w * (S - (p0 + u)); };
  for (int p : da) pl->a.push_back(ModBlock{static_cast<uint16_t>(lo_of(p, 1)), static_cast<uint8_t>(w),
                                            static_cast<uint8_t>(types), 0, 0, 0});
  for (int q : db) pl->b.push_back(ModBlock{static_cast<uint16_t>(lo_of(q, 1)), static_cast<uint8_t>(w),
                                            static_cast<uint8_t>(types), 0, 0, 0});
  pl->pa = static_cast<int>(da.size()) * types;
  pl->pb = static_cast<int>(db.size()) * types;
  pl->direct_bits = w;
  std::map<std::tuple<int, int, int>, int> ablk, bblk;  // (p0, u, moduli) -> first panel
  auto panel_of = [&](std::map<std::tuple<int, int, int>, int>* m, std::vector<ModBlock>* v, int* np, int p0, int u,
                      int nm, bool scaled) {
    const auto key = std::make_tuple(p0, u, nm);
    auto it = m->find(key);
    if (it != m->end()) return it->second;
    v->push_back(ModBlock{static_cast<uint16_t>(lo_of(p0, u)), static_cast<uint8_t>(w * u), static_cast<uint8_t>(nm),
                          1, static_cast<uint8_t>(scaled), 0});
    const int first = *np;
    *np += nm;
    (*m)[key] = first;
    return first;
  };
  struct Seg {
    int a, b;
  };
  for (auto& kv : by) {
    std::vector<Rect>& rs = kv.second;
    const bool direct = std::get<0>(kv.first) == 0;
    std::sort(rs.begin(), rs.end(), [](const Rect& x, const Rect& y) { return x.p < y.p; });
    const int level = std::get<1>(kv.first);
    // operands are at most 128 in magnitude: |sum| <= 2^14 terms, below 2^29 for the
    // residues (the epilogue's division is exact there) and 2^30 for int32 sums
    const int64_t room = (int64_t{1} << (direct ? 16 : 15)) / std::max<int64_t>(k, 1);
    if (room < 1) return false;
    size_t i = 0;
    while (i < rs.size()) {
      // a run of rectangles whose panels advance by constant steps
      const size_t most = std::min(rs.size(), i + static_cast<size_t>(std::min<int64_t>(room, longest)));
      std::vector<Seg> segs;
      size_t j = i;
      int count = types;
      if (direct) {
        for (; j < most; ++j) {
          const int ia = static_cast<int>(std::find(da.begin(), da.end(), rs[j].p) - da.begin());
          const int ib = static_cast<int>(std::find(db.begin(), db.end(), rs[j].q) - db.begin());
          const Seg s{ia * types, ib * types};
          if (segs.size() >= 2 && (s.a - segs.back().a != segs[1].a - segs[0].a ||
                                   s.b - segs.back().b != segs[1].b - segs[0].b))
            break;
          segs.push_back(s);
        }
      } else {
        // up to two rectangles per group: any two are a run
        j = std::min(most, i + 2);
        count = moduli_for(w * (rs[i].u + rs[i].v), static_cast<double>(k) * static_cast<double>(j - i));
        if (count == 0) return false;
        for (size_t x = i; x < j; ++x)
          segs.push_back(Seg{panel_of(&ablk, &pl->a, &pl->pa, rs[x].p, rs[x].u, count, true),
                             panel_of(&bblk, &pl->b, &pl->pb, rs[x].q, rs[x].v, count, false)});
      }
      const int unit = direct ? 4 : 1;
      ModGroup g{};
      g.shift = static_cast<uint16_t>(w * (T - level));
      g.out = static_cast<uint16_t>(pl->planes);
      g.residue = direct ? 0 : 1;
      g.count = static_cast<uint8_t>(count);
      pl->groups.push_back(g);
      const int sa = segs.size() > 1 ? segs[1].a - segs[0].a : 0, sb = segs.size() > 1 ? segs[1].b - segs[0].b : 0;
      for (int x = 0; x < count; ++x) {
        ModJob job{};
        job.a = static_cast<uint16_t>(segs[0].a + x);
        job.b = static_cast<uint16_t>(segs[0].b + x);
        job.da = static_cast<int16_t>(sa);
        job.db = static_cast<int16_t>(sb);
        job.nseg = static_cast<uint16_t>(segs.size());
        job.mod = static_cast<uint16_t>(direct ? kDirectJob : x);
        job.out = static_cast<uint16_t>(pl->planes + x * unit);
        pl->jobs.push_back(job);
        pl->products += static_cast<int64_t>(segs.size());
      }
      (direct ? pl->directs : pl->channels) += direct ? count : (count + 15) / 16;
      pl->planes += count * unit;
      i = j;
      if (pl->pa > kModMaxPanels || pl->pb > kModMaxPanels || pl->planes > 4096 ||
          pl->jobs.size() > static_cast<size_t>(kModMaxJobs) || pl->groups.size() > static_cast<size_t>(kModMaxGroups))
        return false;
    }
  }
  if (pl->a.size() > static_cast<size_t>(kModMaxBlocks) || pl->b.size() > static_cast<size_t>(kModMaxBlocks))
    return false;
  // longest jobs first
  std::stable_sort(pl->jobs.begin(), pl->jobs.end(),
                   [](const ModJob& x, const ModJob& y) { return x.nseg > y.nseg; });
  return true;
}

// kCover: the cost that covers are compared by, from the rates alone.  kPath: the time
// that the product is compared with the other paths by, fitted together with the latencies
// that the caller adds (modular_time_us): one job alone on a CU takes 0.7 of its time
// beside others, a panel byte 0.2 ps besides what every limb read takes.
enum class Estimate { kCover, kPath };
double estimate(const ModPlan& pl, int64_t m, int64_t n, int64_t k, Estimate what) {
  const double alone = what == Estimate::kPath ? 0.7 : 1.0;
  const double panel_byte = what == Estimate::kPath ? 0.7 * kPanelByte : kPanelByte;
  const double mt = static_cast<double>(mod_rows(m)), nt = static_cast<double>(mod_rows(n));
  const double mn = static_cast<double>(m) * static_cast<double>(n);
  // the products: the larger of all blocks spread over the CUs and the longest one
  double s = 0.0, longest = 0.0;
  for (const ModJob& j : pl.jobs) {
    const double block = 2.0 * static_cast<double>(mod_kp(k)) * j.nseg / kInt8Rate + kTileJob;
    s += mt * nt * block;
    longest = std::max(longest, alone * 256.0 * 65536.0 * block);
  }
  s = std::max(s, longest);
  for (const ModJob& j : pl.jobs) s += mn * (j.mod == kDirectJob ? 8.0 / kPlaneRate : 2.0 / kPlaneRate + 0.3e-12);
  return s + panel_byte * static_cast<double>(k) * (static_cast<double>(m) * pl.pa + static_cast<double>(n) * pl.pb);
}

}  // namespace

LevelPlan level_plan(int S, int T, int w) {
  LevelPlan lp;
  lp.S = S;
  lp.T = T;
  lp.c = sub_digits(w);
  for (int i = 0; i < lp.c; ++i)
    for (int p = 0; p < S; ++p) {
      ModBlock b{};
      b.bits = static_cast<uint8_t>(w);
      b.count = 1;
      b.scaled = i == lp.c - 1;
      b.pick = static_cast<uint8_t>(i + 1);
      b.lo = static_cast<uint16_t>(w * (S - 1 - p));
      lp.a.push_back(b);
      b.lo = static_cast<uint16_t>(w * p);  // position p of B's run is digit S - 1 - p
      lp.b.push_back(b);
    }
  return lp;
}

std::shared_ptr<const ModPlan> modular_plan(int64_t m, int64_t n, int64_t k, int S, int T, int w) {
  if (m < 1 || n < 1 || k < 1 || S < 1 || S > kMaxSlices || T < 0 || T > 2 * S - 2 || w < 1 || w > kMaxSliceBits ||
      k > (int64_t{1} << 16))
    return nullptr;
  // shapes enter by powers of sqrt(2), so that nearby products share a cover; k is
  // rounded up, so that the cover's sums stay exact for every k that shares it
  auto code = [](int64_t x) { return static_cast<int>(std::lround(2.0 * std::log2(static_cast<double>(x)))); };
  const int mcode = code(m), ncode = code(n), kcode = static_cast<int>(std::ceil(2.0 * std::log2(k) - 1e-9));
  struct Cache {
    std::mutex mu;
    std::map<std::tuple<int, int, int, int, int, int>, std::shared_ptr<const ModPlan>> map;
  };
  static Cache cache;
  const auto key = std::make_tuple(S, T, w, mcode, ncode, kcode);
  {
    std::lock_guard<std::mutex> lock(cache.mu);
    auto it = cache.map.find(key);
    if (it != cache.map.end()) return it->second;
  }
  const int64_t mc = std::lround(std::exp2(0.5 * mcode)), nc = std::lround(std::exp2(0.5 * ncode));
  const int64_t kc = static_cast<int64_t>(std::ceil(std::exp2(0.5 * kcode) - 1e-6));
  const int c = sub_digits(w), types = c * (c + 1) / 2;
  const double product = 2.0 * static_cast<double>(mod_kp(kc)) / kInt8Rate;
  const double panel = kPanelByte * static_cast<double>(kc) * (1.0 / mc + 1.0 / nc);
  std::shared_ptr<ModPlan> best;
  double least = 0.0;
  for (int residues = 0; residues < 2; ++residues) {
    // the search grows with S^4: the longest operands are covered directly
    if (residues && S > 36) continue;
    std::vector<Rect> rects;
    if (residues) {
      Coverer(S, w, static_cast<double>(kc), product, panel, types).rects(S, S, T, 0, 0, &rects);
    } else {
      for (int p = 0; p < S; ++p)
        for (int q = 0; q < S && p + q <= T; ++q) rects.push_back(Rect{p, q, 1, 1});
    }
    // a level's pairs in one job, or at most two: where the launch leaves CUs idle the
    // longest job is its time
    for (int64_t longest : {int64_t{255}, int64_t{2}}) {
      auto pl = std::make_shared<ModPlan>();
      if (!build(rects, longest, kc, S, T, w, pl.get()) || !modular_accum_fits(*pl, w)) continue;
      const double cost = estimate(*pl, mc, nc, kc, Estimate::kCover);
      if (best && cost >= least) continue;
      least = cost;
      best = pl;
    }
  }
  if (best) best->seconds = estimate(*best, mc, nc, kc, Estimate::kPath);
  std::lock_guard<std::mutex> lock(cache.mu);
  if (cache.map.size() > 4096) cache.map.clear();
  return cache.map.emplace(key, best).first->second;
}

}  // namespace mdg
