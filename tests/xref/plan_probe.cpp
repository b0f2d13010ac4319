// Prints the plans of ising_plan.cpp: reads lines "kind n cus count L...",
// prints "sweep_us tasks count" and, per lattice, "rows strips ls pass threads
// sweeps lds" (count 0: no plan).
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
    const ising::BlockPlan p = ising::plan_blocks(kind, Ls, n, cus);
    std::printf("%.6f %lld %zu", p.sweep_s * 1e6, (long long)p.tasks, p.shapes.size());
    for (const auto& s : p.shapes)
      std::printf(" %d %d %d %d %d %d %zu", s.rows, s.strips, s.ls, s.pass, s.threads, s.sweeps,
                  s.lds);
    std::printf("\n");
  }
  return 0;
}
