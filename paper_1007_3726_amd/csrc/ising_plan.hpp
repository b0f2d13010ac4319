// Plans of the block form: how lattices are cut into strips of rows that take
// several sweeps per launch, and the model that chooses the cut (host part:
// plain C++, no HIP).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace ising {

inline int64_t words_per_row(int64_t L) { return ((L / 2) + 63) / 64; }

inline size_t plane_bytes(int64_t L) {
  return (size_t)L * (size_t)words_per_row(L) * sizeof(uint64_t);
}

// Sweeps of one launch are bounded by the E/M partials of the scratch area:
// 2 slots x kBlockMaxK sweeps x strips x 8 bytes, strips <= kBlockMaxStrips.
constexpr int kBlockMaxK = 16;
constexpr int kBlockMaxStrips = 256;
// Strips of a batch (beyond one per lattice).
constexpr int64_t kBlockMaxTasks = 1024;
// Largest side whose sweeps may take this form with several strips.
constexpr int64_t kBlockMaxL = 16384;
// LDS of one workgroup (two planes of the strip's rows and its halos) where
// two share a compute unit.
constexpr int64_t kBlockMaxLds = 65536;

// Dynamics of a block; kBlockCompare: Philox at thresholds without a cut, for
// plans.
enum { kBlockCompare = -1, kBlockPhilox = 0, kBlockLcg = 1, kBlockPool = 2, kBlockPoolLinear = 3 };

constexpr int kMaxWaves = 16;  // of one workgroup
constexpr int kEmSlots = 32;   // sweeps whose counts are kept in LDS at a time
// 256-word groups of a linear pool that one strip may span.
constexpr int kMaxGroups = 64;
// LDS that the kernels take beside the rows: a pair of counts per sweep and
// wave, and for generators and pools (one kernel) two starts per group.
constexpr int64_t block_static_lds(int kind) {
  return 8 * kEmSlots * kMaxWaves + (kind <= kBlockPhilox ? 0 : 2 * 4 * kMaxGroups);
}
// Rows of a strip that has a compute unit of its own: all that is left.
constexpr int64_t block_lone_lds(int kind) { return 160 * 1024 - block_static_lds(kind); }

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
// Sweeps of a call beyond which strips are not taken: their launches are counted
// in 32 bits, one per sweep at the least.
constexpr int64_t kBlockMaxSweeps = int64_t(1) << 30;
// Calls of at least this many sweeps are all cut alike.
constexpr int64_t kBlockPlanN = 24;
// Distinct sides up to which each is planned by itself, however few the sweeps.
constexpr size_t kBlockPlanSides = 24;

// The cut of a set of lattices (one shape each, in order).
struct BlockPlan {
  std::vector<BlockShape> shapes;  // empty: the set has none
  int32_t sweeps = 0;              // per launch
  int64_t tasks = 0;               // strips in all
  bool all_single = false;         // every lattice in one strip: all sweeps in one launch
  double sweep_s = 0.0;            // model: seconds per sweep of the set
};

BlockShape block_shape_single(int kind, int64_t L);
// Launches of a lattice's n sweeps; one_launch: a single strip runs them all in
// its first launch, else as many per launch as the shape's.
int64_t block_launches(const BlockShape& s, int64_t n, bool one_launch);
// Both planes of a single strip fit one workgroup's LDS.
bool block_fits_single(int64_t L);
// Model: seconds per sweep of lattices with `words` words per colour in all
// when every colour step is a launch.
double launch_per_step_seconds(int kind, double words, int cus);
// The cheapest cut for calls of n sweeps into at most max_tasks strips; empty if
// none takes less than `limit` seconds per sweep.
BlockPlan plan_blocks(int kind, const std::vector<int64_t>& Ls, int64_t n, int cus,
                      double limit = 1e9, int64_t max_tasks = INT64_MAX);

}  // namespace ising
