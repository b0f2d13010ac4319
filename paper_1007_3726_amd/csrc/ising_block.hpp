// Several sweeps per launch on rows held in LDS (ising_block.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "ising_device.hpp"

namespace ising {

// Sweeps of one launch are bounded by the E/M partials of the scratch area:
// 2 slots x kBlockMaxK sweeps x strips x 8 bytes, strips <= kBlockMaxStrips.
constexpr int kBlockMaxK = 16;
constexpr int kBlockMaxStrips = 256;
// Strips of a batch (beyond one per lattice).
constexpr int64_t kBlockMaxTasks = 1024;
// Largest side whose sweeps may take this form with several strips.
constexpr int64_t kBlockMaxL = 16384;
// LDS of one workgroup (two planes of the strip's rows and its halos): half
// of a compute unit's, and where each has a strip of its own nearly all.
constexpr int64_t kBlockMaxLds = 65536;
constexpr int64_t kBlockLoneLds = 156 * 1024;

// Dynamics of a block.
enum { kBlockPhilox = 0, kBlockLcg = 1, kBlockPool = 2, kBlockPoolLinear = 3 };

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

// How one lattice is cut: rows per strip, strips and sweeps per launch.
struct BlockShape {
  int32_t rows = 0, strips = 0, ls = 1, pass = 0, threads = 0, sweeps = 0;
  size_t lds = 0;
  double step_s = 0.0;   // model: seconds of a mean colour step of one strip alone on a CU
  double issue_s = 0.0;  // of which its CU's SIMDs issue for it
  double move_s = 0.0;   // seconds to load and store one strip
};

// Sites of a batch above which it is not worth planning: its colour steps
// take several launches' time.
constexpr double kBlockMaxSites = 6.4e7;
// Calls of at least this many sweeps are all cut alike.
constexpr int64_t kBlockPlanN = 24;

// The cut of a set of lattices (one shape each, in order).
struct BlockPlan {
  std::vector<BlockShape> shapes;  // empty: the set has none
  int32_t sweeps = 0;              // per launch
  int64_t tasks = 0;               // strips in all
  bool all_single = false;         // every lattice in one strip: all sweeps in one launch
  double sweep_s = 0.0;            // model: seconds per sweep of the set
};

}  // namespace ising
