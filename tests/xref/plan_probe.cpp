// Prints the plans of ising_plan.cpp: reads lines "kind n cus count L...",
// prints "plan_us sweep_us tasks count" and, per lattice, "rows strips ls pass
// threads sweeps lds" (count 0: no plan), and 1 if that is cheaper than a launch
// per colour step.  plan_us: microseconds that the planning of several
// lattices takes when it is held to that, the best of three.
#include <chrono>
#include <cstdio>

#include "ising_plan.hpp"

int main() {
  int kind, cus, count;
  long long n;
  while (std::scanf("%d %lld %d %d", &kind, &n, &cus, &count) == 4) {
    std::vector<int64_t> Ls;
    for (int i = 0; i < count; ++i) {
      long long L;
      if (std::scanf("%lld", &L) != 1) return 1;
      Ls.push_back(L);
    }
    double words = 0, us = 1e9;
    for (int64_t L : Ls) words += (double)(L * ising::words_per_row(L));
    for (int i = 0; i < 3 && count > 1; ++i) {
      const auto t0 = std::chrono::steady_clock::now();
      ising::plan_blocks(kind, Ls, n, cus, ising::launch_per_step_seconds(kind, words, cus));
      const std::chrono::duration<double, std::micro> d = std::chrono::steady_clock::now() - t0;
      if (d.count() < us) us = d.count();
    }
    const ising::BlockPlan p = ising::plan_blocks(kind, Ls, n, cus);
    std::printf("%.3f %.6f %lld %zu", us, p.sweep_s * 1e6, (long long)p.tasks, p.shapes.size());
    for (const auto& s : p.shapes)
      std::printf(" %d %d %d %d %d %d %zu", s.rows, s.strips, s.ls, s.pass, s.threads, s.sweeps,
                  s.lds);
    std::printf(" %d\n", !p.shapes.empty() &&
                              p.sweep_s < ising::launch_per_step_seconds(kind, words, cus));
  }
  return 0;
}
