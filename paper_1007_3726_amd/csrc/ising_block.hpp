// Several sweeps per launch on rows held in LDS (ising_block.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"
#include "ising_plan.hpp"

namespace ising {

struct BlockAlt {
  int32_t kind;
  uint32_t* lcg;         // generators [2][L][W]
  const uint64_t* pool;  // (r4, r8) pairs
  uint32_t pool_shift, pool_mask;
};

struct BlockLattice {
  uint64_t* buf[2];    // planes; several strips: launch j reads buf[j & 1], writes the other
  int32_t L, W, half;  // side, words per row, sites of a colour row
  int32_t nh, nbl;     // 32-bit halves per row, valid bits of the last one
  int32_t rows;        // rows per strip (L for a single strip)
  int32_t strips;
  int32_t ls;          // lanes per half: 1, 2, 4 or 8; 0: a lane per word (pools)
  int32_t pass;        // rows per pass of the workgroup
  int32_t threads;     // pass * nh * ls, rounded up to whole waves
  int32_t launches;    // launches that this lattice's n sweeps are dealt over
  uint32_t k0, k1, sid4, t, t4, t8;
  Cut cut;
  int64_t n;           // sweeps in all
  int64_t* EM;         // n x 2 per-sweep (E, M), or null
  uint32_t* part;      // several strips: E/M partials
  uint32_t perturb;    // test hook: nonzero seeds pauses before block barriers
};

struct BlockTask {
  int32_t lattice, strip;
};

}  // namespace ising
