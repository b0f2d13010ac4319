// Plans of the block form (ising_plan.hpp): plain C++, no HIP.
#include "ising_plan.hpp"

#include <algorithm>
#include <cmath>
#include <functional>
#include <utility>

namespace ising {

// Measured costs of the model below, in cycles and seconds.
constexpr double kClock = 2.4e9;
constexpr double kLaunch = 5e-6;   // a launch: gap, loads, stores
constexpr double kBarrier = 1e-7;  // of a colour step
constexpr double kCuBytes = 2.5e10;  // bytes per second of one compute unit's share
constexpr double kPatternLatency = 1e-6;
constexpr double kAdvance = 3.5e-6;  // generators moved on, once per call

// Instructions of one wave's pass with ls lanes per half; `any`: rows that
// start anywhere in a Philox block.
static double pass_instructions(int kind, int ls, bool any) {
  if (kind == kBlockLcg) return ls == 8 ? 85 : ls == 4 ? 105 : ls == 2 ? 140 : 210;
  if (kind == kBlockPool) return ls == 0 ? 165 : 115;
  if (kind == kBlockPoolLinear) return ls == 0 ? 105 : 75;
  // (four and eight lanes compare anyway)
  const double more = kind == kBlockCompare && ls <= 2 ? 1.13 : 1.0;
  if (any) return more * (ls == 8 ? 155 : ls == 4 ? 220 : ls == 2 ? 335 : 515);
  return more * (ls == 8 ? 115 : ls == 4 ? 180 : ls == 2 ? 290 : 460);
}

static double waves_of(double halves, int ls) { return std::ceil(halves * (ls ? ls : 0.5) / 64); }

// Seconds of one colour step of a workgroup that updates `halves` halves with
// the compute unit to itself: the busiest SIMD issues its waves' instructions
// one per four cycles, and a lone wave no more than one per six.
static double step_seconds(int kind, double halves, int ls, bool any) {
  const double issue = std::ceil(waves_of(halves, ls) / 4) * 4, alone = 6;
  double s = std::max(issue, alone) * pass_instructions(kind, ls, any) / kClock + kBarrier;
  // patterns: one load's latency, and 8 bytes per half at a CU's share of the
  // memory's rate (a 128-byte line per random pattern)
  if (kind == kBlockPoolLinear) s = std::max(s, halves * 8 / kCuBytes) + kPatternLatency;
  if (kind == kBlockPool) s = std::max(s, halves * 64 / kCuBytes) + kPatternLatency;
  return s;
}

// Strips of `rows` rows with K sweeps per launch.
static BlockShape shape_of(int kind, int64_t L, int64_t rows, int K, int max_ls = 8) {
  BlockShape s;
  const int64_t W = words_per_row(L), nh = (L / 2 + 31) / 32;
  const bool single = rows >= L, any = L % 8 != 0;
  s.rows = (int32_t)std::min(rows, L);
  s.strips = single ? 1 : (int32_t)((L + rows - 1) / rows);
  s.sweeps = K;
  const int64_t R = single ? L : s.rows + 4 * (int64_t)K;       // rows in LDS
  const int64_t mean = single ? L : s.rows + 2 * (int64_t)K;    // rows of a mean step
  // More lanes per half make more waves of fewer instructions, but more
  // instructions in all (115 / 256, 290 / 1024, 460 / 2048 sites): as many
  // lanes as shorten the step.  Measured, us per sweep with 1, 2, 4, 8 lanes:
  // 64^2 1.71, 1.09, 0.92, 0.93; 128^2 1.90, 1.92, 2.17, 3.69; 512^2 in strips
  // of 2 rows, 8 sweeps 2.84, 2.66, 2.79, 3.07; 2048^2 in strips of 8 rows, 4
  // sweeps 5.34, 5.57, 6.23, 7.96.
  const double halves = (double)(mean * nh);
  s.ls = 1;
  s.step_s = step_seconds(kind, halves, 1, any);
  auto offer = [&](int ls) {
    const double step = step_seconds(kind, halves, ls, any);
    if (step < s.step_s) {
      s.ls = ls;
      s.step_s = step;
    }
  };
  for (int ls = 2; ls <= max_ls && kind <= kBlockLcg && nh * ls <= 1024; ls *= 2) offer(ls);
  // pools: a whole word per lane (ls 0) where that leaves enough waves: a lone
  // wave's step is longer with it (64^2, 128^2 stay with halves)
  if (kind >= kBlockPool) offer(0);
  const int64_t per = s.ls ? nh * s.ls : W;
  s.pass = (int32_t)std::max<int64_t>(1, std::min<int64_t>(R, 1024 / per));
  s.threads = (int32_t)((s.pass * per + 63) / 64 * 64);
  s.lds = (size_t)(R * W) * (kind == kBlockLcg ? 24 : 16);
  s.issue_s = waves_of(halves, s.ls) * pass_instructions(kind, s.ls, any) / kClock;
  s.move_s = (double)(s.lds + 16 * s.rows * W) / kCuBytes;
  return s;
}

// Measured: 3 us per launch (gap, ramp and drain) and 1.45 us per word of the
// busiest SIMD's waves, at least 2.2 us for a word alone: us per sweep 15.3 at
// 4104^2, 20.7 at 6000^2, 29.3 at 8192^2, 74 for the 56-lattice grid.  Without a
// cut of the thresholds 1.645 us, against 1.13 of the blocks' instructions: 16
// sweeps of 6144^2 at T = 1.5 22.5 us each in tiles, 23.4 in blocks (at 2.3 20.5
// and 20.7).  Generators 0.58 us and 1.5 us (their chain is serial), patterns
// 0.35 us (random 1.4 us) and 1 us: 16384^2 24.0, 14.2 and 45.7 us per colour
// step.
double launch_per_step_seconds(int kind, double words, int cus) {
  static const double word[] = {1.645e-6, 1.45e-6, 0.65e-6, 1.35e-6, 0.35e-6};
  static const double alone[] = {2.2e-6, 2.2e-6, 1.5e-6, 1.0e-6, 1.0e-6};
  const int k = kind - kBlockCompare;
  return 2 * (3e-6 + std::max(alone[k], word[k] * std::ceil(words / 256 / std::max(cus, 1))));
}

BlockShape block_shape_single(int kind, int64_t L) { return shape_of(kind, L, L, 1); }

int64_t block_launches(const BlockShape& s, int64_t n, bool one_launch) {
  if (s.strips == 1) {
    const int64_t per = one_launch ? (int64_t)1 << 20 : s.sweeps;
    return std::max<int64_t>((n + per - 1) / per, 1);
  }
  // an even number of launches leaves the result in the lattice's own planes
  return 2 * ((n + 2 * s.sweeps - 1) / (2 * s.sweeps));
}

// Both planes of a single strip fit one workgroup's LDS.
bool block_fits_single(int64_t L) {
  return L <= kBlockMaxL && 2 * (int64_t)plane_bytes(L) <= kBlockMaxLds;
}

// Issue time of a colour step on the busiest compute unit: the strips go out
// from the largest down, so that it has the first, the first after all units
// have one, and so on.  A queue of 24 requests up to 2048^2: 28.9 ms with 379
// strips, the best if they spread evenly over 256 units, 25.7 ms this way.
static double busiest_issue(const std::vector<BlockShape>& shapes,
                            const std::vector<std::pair<int64_t, int64_t>>& sides, int cus,
                            std::vector<std::pair<double, int64_t>>& of) {
  of.clear();
  for (size_t i = 0; i < shapes.size(); ++i)
    of.push_back({shapes[i].issue_s, shapes[i].strips * sides[i].second});
  std::sort(of.rbegin(), of.rend());
  double sum = 0;
  int64_t seen = 0, next = 0;  // strips so far; the unit's next strip
  for (const auto& o : of)
    for (seen += o.second; next < seen; next += std::max(cus, 1)) sum += o.first;
  return sum;
}

// A set of lattices to be cut, and the cheapest cut found so far.
namespace {
typedef std::vector<std::pair<int64_t, int64_t>> Sides;  // (side, lattices), largest first

struct CutOf {  // sweeps per launch, halves per strip, lanes; target 0: one strip each
  int K = 0;
  int64_t target = 0;
  int max_ls = 8;
};

struct Search {
  int kind;
  Sides sides;
  int64_t lattices, lds, most;  // most: strips
  int cus;
  int64_t n;          // sweeps per call
  BlockPlan best, p;  // a shape per side
  CutOf cut;           // best's
  std::vector<std::pair<double, int64_t>> of;

  Search(int kind_, const Sides& sides_, int64_t lattices_, int cus_, int64_t n_, double limit,
         int64_t max_tasks)
      : kind(kind_), sides(sides_), lattices(lattices_), cus(cus_), n(n_) {
    most = std::min(kBlockMaxTasks + lattices, max_tasks);
    // a lone lattice's strips have a compute unit each
    lds = lattices == 1 ? block_lone_lds(kind) : kBlockMaxLds;
    best.sweep_s = limit;
  }

  void consider(const CutOf& c) {
    const bool singles = c.target == 0;
    const int K = c.K;
    // launches per sweep of a lattice of several strips
    const bool few = few_sweeps();
    const double per = few ? (double)(2 * ((n + 2 * K - 1) / (2 * K))) / n : 1.0 / K;
    const double call = few && kind == kBlockLcg ? kAdvance / n : 0.0;
    const double fixed = (singles ? 0.0 : kLaunch * per) + call, units = std::max(cus, 1);
    double longest = 0, move = 0, issue = 0;
    int64_t strips = 0;
    p.shapes.clear();
    for (const auto& side : sides) {
      const int64_t L = side.first, nh = (L / 2 + 31) / 32;
      // L rows at most in LDS, kBlockMaxStrips strips at most
      int64_t rows = std::max<int64_t>(c.target / nh - 2 * (int64_t)K, 1);
      rows = std::max(rows, (L + kBlockMaxStrips - 1) / kBlockMaxStrips);
      const bool single = block_fits_single(L) && (singles || rows + 2 * K >= L);
      // (with the largest side all others are single: one launch is cheaper)
      if (single && !singles && p.shapes.empty()) return;
      if (single)
        rows = L;
      else if (singles || rows + 4 * (int64_t)K > L)
        return;
      const BlockShape s = shape_of(kind, L, rows, K, c.max_ls);
      if (s.lds > (size_t)lds || (!single && K > s.strips)) return;
      if (kind == kBlockPoolLinear && (int64_t)(s.lds / 16) / 256 + 3 > kMaxGroups) return;
      strips += s.strips * side.second;
      if (strips > most) return;
      longest = std::max(longest, s.step_s);
      issue += s.issue_s * (double)(s.strips * side.second);
      // no cheaper than the best even if no other strip is longer and all of
      // them spread evenly (the busiest unit has the mean at least)
      if (2 * std::max(longest, issue / units) + fixed >= best.sweep_s) return;
      p.shapes.push_back(s);
      move = std::max(move, s.move_s);
    }
    p.sweeps = K;
    p.tasks = strips;
    const double step = std::max(longest, busiest_issue(p.shapes, sides, cus, of));
    p.sweep_s = 2 * step + fixed + (singles ? 0.0 : move * per);
    if (p.sweep_s < best.sweep_s) {
      std::swap(best, p);
      cut = c;
    }
  }

  // A call of few sweeps counts its launches one by one: they share the sweeps
  // evenly (5 sweeps: 3 and 2, or 2, 1, 1, 1), and generators have one of their
  // own.  As if every launch had K sweeps, calls of 2 to 8 sweeps took blocks
  // where tiles are up to 13 % faster (5 sweeps of 4002^2 13.3 and 15.0 us each),
  // or too many launches (1400^2 6.5 -> 5.2).  Pools stay with that: their steps
  // cost less than the model has them at, and counted so they would be left to
  // tiles that are up to 40 % slower.
  bool few_sweeps() const { return n < kBlockPlanN && kind <= kBlockLcg; }

  std::vector<int> sweeps_per_launch() const {
    std::vector<int> Ks;
    if (!few_sweeps()) {
      for (int K : {1, 2, 3, 4, 6, 8, 12})
        if (K <= (n + 1) / 2) Ks.push_back(K);
      return Ks;
    }
    for (int64_t K = 1; K <= (n + 1) / 2; ++K) {
      const int64_t m = 2 * ((n + 2 * K - 1) / (2 * K));
      if ((n + m - 1) / m == K) Ks.push_back((int)K);
    }
    return Ks;
  }

  // With more lattices than compute units a lattice's own
  // step counts for less than the instructions in all, so that fewer lanes per
  // half can win: 300 sweeps of 600 lattices of 64^2 3.3 -> 1.1 ms, of 128^2
  // 5.3 -> 1.95.
  void all() {
    const int least = lattices > cus ? 1 : 8;
    for (int max_ls = 8; max_ls >= least; max_ls /= 2) consider(CutOf{1, 0, max_ls});
    if (n < 2) return;
    std::vector<int64_t> targets;
    for (int64_t target = 32; target <= 20000; target += target / 4) targets.push_back(target);
    // every fourth target first, so that the others are measured by a good cut
    const std::vector<int> Ks = sweeps_per_launch();
    for (size_t step : {4, 1})
      for (int max_ls = 8; max_ls >= least; max_ls /= 2)
        for (int K : Ks)
          for (size_t i = 0; i < targets.size(); i += step)
            if (step == 4 || i % 4) consider(CutOf{K, targets[i], max_ls});
  }
};

// Runs of neighbouring sides as so many of their middle one: few enough to be
// searched in the time of a few sweeps.
Sides grouped(const Sides& sides) {
  const size_t run = (sides.size() + kBlockPlanSides - 1) / kBlockPlanSides;
  Sides g;
  for (size_t at = 0; at < sides.size(); at += run) {
    const size_t end = std::min(at + run, sides.size());
    g.push_back({sides[(at + end) / 2].first, 0});
    for (size_t i = at; i < end; ++i) g.back().second += sides[i].second;
  }
  return g;
}
}  // namespace

// The cheapest cut of a set of lattices by the model: sweeps per launch K,
// and strips of about `target` halves per mean colour step, so that the
// strips of all lattices are about equal.  A lattice that fits one workgroup
// takes a single strip where a strip would be as large.  The host waits for
// this in every batched call, so a cut is given up as soon as it cannot win,
// and with many sides and few sweeps near sides are searched as one.  A call
// of 24 sweeps of 24, 87 or 120 distinct sides is planned in 0.06, 0.10 and
// 0.14 ms, 0.34, 1.8 and 10.5 with every cut of every side.
BlockPlan plan_blocks(int kind, const std::vector<int64_t>& Ls, int64_t n, int cus,
                      double limit, int64_t max_tasks) {
  std::vector<int64_t> sorted(Ls);
  std::sort(sorted.begin(), sorted.end(), std::greater<int64_t>());
  Sides sides;
  for (int64_t L : sorted) {
    if (sides.empty() || sides.back().first != L) sides.push_back({L, 0});
    ++sides.back().second;
  }
  const int64_t lattices = (int64_t)Ls.size();
  Search s(kind, sides, lattices, cus, n, limit, max_tasks);
  // (grouped, a cut is up to a tenth dearer: 87 sides 12.5 us per sweep, each
  // by itself 11.6, in four times the planning)
  if (sides.size() <= kBlockPlanSides || n >= 8 * (int64_t)sides.size()) {
    s.all();
  } else {
    // the cut of the groups, with strips as long and around that
    Search g(kind, grouped(sides), lattices, cus, n, 1.1 * limit, max_tasks);
    g.all();
    if (g.best.shapes.empty()) return BlockPlan();
    s.consider(g.cut);
    for (double f : {1.25, 0.8, 1.5, 0.65, 1.9})
      if (g.cut.target)
        s.consider(CutOf{g.cut.K, (int64_t)(f * (double)g.cut.target), g.cut.max_ls});
    if (s.best.shapes.empty()) s.all();
  }
  BlockPlan best;
  if (s.best.shapes.empty()) return best;
  best = s.best;
  std::vector<BlockShape> shapes;
  best.all_single = true;
  for (int64_t L : Ls) {
    const auto at = std::lower_bound(
        sides.begin(), sides.end(), L,
        [](const std::pair<int64_t, int64_t>& side, int64_t v) { return side.first > v; });
    shapes.push_back(best.shapes[at - sides.begin()]);
    best.all_single = best.all_single && shapes.back().strips == 1;
  }
  best.shapes = shapes;
  return best;
}

}  // namespace ising
