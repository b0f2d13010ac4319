// Plans of the block form (ising_plan.hpp): plain C++, no HIP.
#include "ising_plan.hpp"

#include <algorithm>
#include <cmath>
#include <functional>
#include <iterator>
#include <map>
#include <utility>

namespace ising {

// Measured costs of the model below, in cycles and seconds.
constexpr double kClock = 2.4e9;
constexpr double kLaunch = 5e-6;   // a launch: gap, loads, stores
constexpr double kBarrier = 1e-7;  // of a colour step
constexpr double kCuBytes = 2.5e10;  // bytes per second of one compute unit's share
constexpr double kPatternLatency = 1e-6;

// Instructions of one wave's pass with ls lanes per half; `any`: rows that
// start anywhere in a Philox block.
static double pass_instructions(int kind, int ls, bool any) {
  if (kind == kBlockLcg) return ls == 8 ? 85 : ls == 4 ? 105 : ls == 2 ? 140 : 210;
  if (kind == kBlockPool) return ls == 0 ? 165 : 115;
  if (kind == kBlockPoolLinear) return ls == 0 ? 105 : 75;
  if (any) return ls == 8 ? 155 : ls == 4 ? 220 : ls == 2 ? 335 : 515;
  return ls == 8 ? 115 : ls == 4 ? 180 : ls == 2 ? 290 : 460;
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
  s.ls = 1;
  const double halves = (double)(mean * nh);
  for (int ls = 2; ls <= max_ls && kind <= kBlockLcg; ls *= 2)
    if (nh * ls <= 1024 &&
        step_seconds(kind, halves, ls, any) < step_seconds(kind, halves, s.ls, any))
      s.ls = ls;
  // pools: a whole word per lane (ls 0) where that leaves enough waves: a lone
  // wave's step is longer with it (64^2, 128^2 stay with halves)
  if (kind >= kBlockPool && step_seconds(kind, halves, 0, any) < step_seconds(kind, halves, 1, any))
    s.ls = 0;
  const int64_t per = s.ls ? nh * s.ls : W;
  s.pass = (int32_t)std::max<int64_t>(1, std::min<int64_t>(R, 1024 / per));
  s.threads = (int32_t)((s.pass * per + 63) / 64 * 64);
  s.lds = (size_t)(R * W) * (kind == kBlockLcg ? 24 : 16);
  s.step_s = step_seconds(kind, halves, s.ls, any);
  s.issue_s = waves_of(halves, s.ls) * pass_instructions(kind, s.ls, any) / kClock;
  s.move_s = (double)(s.lds + 16 * s.rows * W) / kCuBytes;
  return s;
}

// Measured: 3 us per launch (gap, ramp and drain) and 1.45 us per word of the
// busiest SIMD's waves, at least 2.2 us for a word alone: us per sweep 15.3 at
// 4104^2, 20.7 at 6000^2, 29.3 at 8192^2, 74 for the 56-lattice grid.
// Generators 0.58 us and 1.5 us (their chain is serial), patterns 0.35 us
// (random 1.4 us) and 1 us: 16384^2 24.0, 14.2 and 45.7 us per colour step.
double launch_per_step_seconds(int kind, double words, int cus) {
  static const double word[] = {1.45e-6, 0.65e-6, 1.35e-6, 0.35e-6};
  static const double alone[] = {2.2e-6, 1.5e-6, 1.0e-6, 1.0e-6};
  return 2 * (3e-6 + std::max(alone[kind], word[kind] * std::ceil(words / 256 / std::max(cus, 1))));
}

BlockShape block_shape_single(int kind, int64_t L) { return shape_of(kind, L, L, 1); }

// Both planes of a single strip fit one workgroup's LDS.
bool block_fits_single(int64_t L) {
  return L <= kBlockMaxL && 2 * (int64_t)plane_bytes(L) <= kBlockMaxLds;
}

// Issue time of a colour step on the busiest compute unit: the strips go out
// from the largest down, so that it has the first, the first after all units
// have one, and so on.  A queue of 24 requests up to 2048^2: 28.9 ms with 379
// strips, the best if they spread evenly over 256 units, 25.7 ms this way.
static double busiest_issue(const std::vector<BlockShape>& shapes,
                            const std::vector<std::pair<int64_t, int64_t>>& sides, int cus) {
  std::vector<std::pair<double, int64_t>> of;
  for (size_t i = 0; i < shapes.size(); ++i)
    of.push_back({shapes[i].issue_s, shapes[i].strips * sides[i].second});
  std::sort(of.rbegin(), of.rend());
  double sum = 0;
  int64_t seen = 0, next = 0;  // strips so far; the unit's next strip
  for (const auto& o : of)
    for (seen += o.second; next < seen; next += std::max(cus, 1)) sum += o.first;
  return sum;
}

// The cheapest cut of a set of lattices by the model: sweeps per launch K,
// and strips of about `target` halves per mean colour step, so that the
// strips of all lattices are about equal.  A lattice that fits one workgroup
// takes a single strip where a strip would be as large.  With more lattices
// than compute units a lattice's own step counts for less than the
// instructions in all, so that fewer lanes per half can win: 300 sweeps of 600
// lattices of 64^2 3.3 -> 1.1 ms, of 128^2 5.3 -> 1.95.
BlockPlan plan_blocks(int kind, const std::vector<int64_t>& Ls, int64_t n, int cus) {
  BlockPlan best;  // a shape per distinct side
  bool all_single = true;
  for (int64_t L : Ls) all_single = all_single && block_fits_single(L);
  std::map<int64_t, int64_t, std::greater<int64_t>> of;
  for (int64_t L : Ls) ++of[L];
  const std::vector<std::pair<int64_t, int64_t>> sides(of.begin(), of.end());
  // a lone lattice's strips have a compute unit each
  const int64_t lds = Ls.size() == 1 ? block_lone_lds(kind) : kBlockMaxLds;
  auto consider = [&](int K, int64_t target, bool singles, int max_ls) {
    BlockPlan p;
    double longest = 0, move = 0;
    int64_t strips = 0;
    for (const auto& side : sides) {
      const int64_t L = side.first, nh = (L / 2 + 31) / 32;
      // L rows at most in LDS, kBlockMaxStrips strips at most
      int64_t rows = std::max<int64_t>(target / nh - 2 * (int64_t)K, 1);
      rows = std::max(rows, (L + kBlockMaxStrips - 1) / kBlockMaxStrips);
      const bool single = block_fits_single(L) && (singles || rows + 2 * K >= L);
      if (single)
        rows = L;
      else if (rows + 4 * (int64_t)K > L)
        return;
      const BlockShape s = shape_of(kind, L, rows, K, max_ls);
      if (s.lds > (size_t)lds || (!single && K > s.strips)) return;
      if (kind == kBlockPoolLinear && (int64_t)(s.lds / 16) / 256 + 3 > kMaxGroups) return;
      // no cheaper than the best even if this strip is the longest (planning
      // 24 lattices took 0.15 ms of the host without this line)
      if (!best.shapes.empty() && 2 * s.step_s + (singles ? 0.0 : kLaunch / K) >= best.sweep_s)
        return;
      p.shapes.push_back(s);
      longest = std::max(longest, s.step_s);
      move = std::max(move, s.move_s);
      strips += s.strips * side.second;
    }
    if (strips > kBlockMaxTasks + (int64_t)Ls.size()) return;
    p.sweeps = K;
    p.tasks = strips;
    const double step = std::max(longest, busiest_issue(p.shapes, sides, cus));
    p.sweep_s = 2 * step + (singles ? 0.0 : (kLaunch + move) / K);
    if (best.shapes.empty() || p.sweep_s < best.sweep_s) best = p;
  };
  for (int max_ls = 8; max_ls >= ((int64_t)Ls.size() > cus ? 1 : 8); max_ls /= 2) {
    if (all_single) consider(1, 0, true, max_ls);
    if (n >= 2)
      for (int K : {1, 2, 3, 4, 6, 8, 12})
        if (K <= (n + 1) / 2)
          for (int64_t target = 32; target <= 20000; target += target / 4)
            consider(K, target, false, max_ls);
  }
  if (best.shapes.empty()) return best;
  std::vector<BlockShape> shapes;
  best.all_single = true;
  for (int64_t L : Ls) {
    shapes.push_back(best.shapes[std::distance(of.begin(), of.find(L))]);
    best.all_single = best.all_single && shapes.back().strips == 1;
  }
  best.shapes = shapes;
  return best;
}

}  // namespace ising
