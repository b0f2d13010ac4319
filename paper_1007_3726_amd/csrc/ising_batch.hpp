// Batched sweeps (internal).
#pragma once

#include <stdint.h>

#include <vector>

#include "ising_runtime.hpp"

namespace ising {

struct BatchOptions {
  int wg_per_cu;    // workgroups per compute unit of the fused grid
  int force_form;   // -1: cost model, 0: fused, 1: packed
  int graph_chunk;  // sweeps per captured hipGraph chunk (0: no graph)
  // row groups per wave of a lattice's tiles: the largest r in {1, 2, 4},
  // r <= rpw_max, for which the lattice has at least 128 r tiles of one row
  // group per wave, of at most kTileMaxWords words each
  int rpw_max = 2;
  // when set (with graph_chunk 0): the table image is kept here, since it
  // must outlive its asynchronous upload, and the call returns without
  // waiting for the stream; the caller synchronises before it reuses the
  // image or the work buffer
  std::vector<char>* keep_image = nullptr;
};

// The built-in batched options, with the batched autotuner's installed
// fused shape (rpw_max, workgroups per CU, graph chunk) if there is one.
BatchOptions default_batch_options();
// Argument checks shared by the batched entry points (n: sweeps to come).
ising_status check_batch(ising_t* const* hs, int32_t count, int64_t n, const char* who);
// Whether these lattices together are cheaper in blocks than in a launch per
// colour step, for n sweeps (the cut in *plan); kind: kBlockPhilox, or
// kBlockCompare where none of them has a cut of its thresholds; table_bytes: room
// for the plan's tables.
bool choose_blocks(int kind, const std::vector<int64_t>& Ls, int64_t n, int cus,
                   size_t table_bytes, BlockPlan* plan);
// Device bytes of the work buffer batch_sweeps needs for these handles
// (0 when every lattice takes the plain path).
size_t batch_work_bytes(ising_lattice* const* hs, int32_t count, const BatchOptions& opt);
// An upper bound of one lattice's share of that buffer, whatever the form
// and the rest of the batch: batch_work_bytes of a set of lattices is at most
// kBatchWorkFixed plus the sum of their shares.
size_t batch_work_share(int64_t L);
constexpr size_t kBatchWorkFixed = 4 * 256;
// Advance hs[i] by nsw[i] sweeps (nsw may be null: n for all), n = max nsw,
// with the task tables in `work` (device, 256-byte aligned, work_bytes >=
// batch_work_bytes).  Does not change the handles' sweep counters.
ising_status batch_sweeps(ising_lattice* const* hs, int32_t count, int64_t n,
                          const int64_t* nsw, int64_t* const* dev_EM, const BatchOptions& opt,
                          void* work, size_t work_bytes, int* form_out);

// Several sweeps per launch (ising_block.hip).
int block_kind(const ising_lattice* h);
// One lattice's entry for n sweeps; one_launch: a single strip runs them all
// in its first launch, else as many per launch as the shape's.
BlockLattice block_lattice(const ising_lattice* h, const BlockShape& s, int64_t n,
                           bool one_launch, int64_t* EM);
ising_status enqueue_block_sweeps(ising_lattice* h, const BlockShape& s, int64_t n,
                                  int64_t* dev_EM);
hipError_t launch_block_many(hipStream_t st, const BlockLattice* tab, const BlockTask* tasks,
                             int ntasks, int cus, int threads, size_t lds, int j);
hipError_t launch_block_finalize_many(hipStream_t st, const BlockLattice* tab, int nlat);
// Compute units of a device (cached), 0 if it has no properties.
int device_cus(int device);

}  // namespace ising
