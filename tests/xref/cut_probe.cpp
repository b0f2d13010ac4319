// Evaluates the three-way cut of ising_cut.hpp on the host: reads lines
// "t4 t8 u_max u", prints "x code" (x = 0: no cut for these thresholds).
#include <cstdio>

#include "ising_cut.hpp"

int main() {
  unsigned t4, t8, top, u;
  while (std::scanf("%u %u %u %u", &t4, &t8, &top, &u) == 4) {
    const ising::Cut c = ising::make_cut(t4, t8, top);
    std::printf("%u %u\n", c.x, (unsigned)(((uint64_t)u * c.x + c.c) >> 60));
  }
  return 0;
}
