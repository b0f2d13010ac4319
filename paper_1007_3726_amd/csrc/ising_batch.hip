// Batched sweeps: many lattices of uneven size and temperature.
//
// Two launch forms, chosen per call by the cost model of the blocks
// (ising_plan.cpp):
//   * fused: the tiles of all lattices form one flat list; each sweep is
//     two launches of k_fused (colour 0, colour 1) that walk the whole list,
//     so every colour step is balanced over the whole GPU.  Long runs are
//     replayed from a captured hipGraph chunk of K sweeps (a device-side
//     sweep counter advanced by the last node keeps the chunk reusable);
//   * blocks (ising_block.hip): several sweeps per launch on rows held in LDS,
//     for batches whose colour steps would not fill the GPU for longer than a
//     launch takes; a batch of lattices that each fit one workgroup ("packed")
//     runs all n sweeps in one launch.
// Lattices the tiled layout does not cover (L % 8 != 0, or Philox block
// indices crossing 2^32 inside a row) are advanced with the plain path unless
// the whole batch takes blocks.
// The task tables live in a work buffer the caller provides (device
// memory, batch_work_bytes of it); the library allocates no device memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>
#include <vector>

#include "ising_batch.hpp"
#include "ising_runtime.hpp"

namespace ising {

bool tile_args(const ising_lattice* h, TileArgs* out);

namespace {

// Per-device host state: the compute-unit count and a private stream for
// graph capture (the caller's stream may be the null stream, which cannot
// be captured).  The mutex serialises captures on that stream.
struct DeviceState {
  std::mutex m;
  std::atomic<int> cus{0};
  hipStream_t capture = nullptr;
};

DeviceState& state_for(int device) {
  static DeviceState states[64];
  return states[device & 63];
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Byte offsets of the fused form's tables in the work buffer.
struct FusedLayout {
  size_t off_k = 0, off_lat = 256, off_tiles = 0, off_part = 0, bytes = 0;
};

FusedLayout fused_layout(size_t nl, size_t ntiles, size_t record = sizeof(FusedLattice)) {
  FusedLayout f;
  f.off_tiles = align_up(f.off_lat + nl * record, 256);
  f.off_part = align_up(f.off_tiles + ntiles * sizeof(FusedTile), 256);
  // per-wave E/M partials: 2 sweep slots x 4 waves x (anti, up) per tile
  f.bytes = align_up(f.off_part + 2 * 4 * 2 * ntiles * sizeof(uint32_t), 256);
  return f;
}

// Byte offsets of the block form's tables.
struct BlockLayout {
  size_t off_tasks = 0, bytes = 0;
};

BlockLayout block_layout(size_t nl, size_t ntasks) {
  BlockLayout p;
  p.off_tasks = align_up(nl * sizeof(BlockLattice), 256);
  p.bytes = align_up(p.off_tasks + ntasks * sizeof(BlockTask), 256);
  return p;
}

// Tiles of the fused form's flat mapping for one lattice (RPW row groups per wave).
int64_t fused_tiles(int64_t plane_words, int32_t rpw) {
  const int64_t per_tile = 256 * (int64_t)rpw;
  return (plane_words + per_tile - 1) / per_tile;
}

int fused_grid(int64_t tiles, int wg_per_cu, int cus) {
  return (int)std::min<int64_t>(std::max<int64_t>(tiles, 1), (int64_t)wg_per_cu * cus);
}

}  // namespace

// Without the mutex: a batch holds that until its captured sweeps are done, and
// every sweep of a lone lattice comes here.
int device_cus(int device) {
  DeviceState& D = state_for(device);
  int cus = D.cus.load(std::memory_order_relaxed);
  if (cus == 0) {
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, device) == hipSuccess) cus = p.multiProcessorCount;
    D.cus.store(cus, std::memory_order_relaxed);
  }
  return cus;
}

// A batch of more sites than kBlockMaxSites fills the chip in every colour
// step: only single strips, which have no halo rows, can still be cheaper.
// (And only they run any number of sweeps.)
bool choose_blocks(int kind, const std::vector<int64_t>& Ls, int64_t n, int cus,
                   size_t table_bytes, BlockPlan* plan) {
  double sites = 0, words = 0;
  bool all_single = true;
  for (int64_t L : Ls) {
    if (L > kBlockMaxL) return false;
    sites += (double)L * L;
    words += (double)(L * words_per_row(L));
    all_single = all_single && block_fits_single(L);
  }
  if (sites > kBlockMaxSites || n > kBlockMaxSweeps) {
    if (!all_single) return false;
    n = 1;
  }
  // a batch of few lattices has tables for fewer strips than the chip has units:
  // 200 sweeps of 3 x 336^2 2.13 ms where the best cut did not fit and the fused
  // form ran, 0.62 with the best that fits
  const size_t off = block_layout(Ls.size(), 0).off_tasks, room = table_bytes / 256 * 256;
  const int64_t most = room > off ? (int64_t)((room - off) / sizeof(BlockTask)) : 0;
  *plan = plan_blocks(kind, Ls, n, cus, launch_per_step_seconds(kind, words, cus), most);
  return !plan->shapes.empty();
}

static ising_status run_fused(ising_lattice* const* hs, const std::vector<int>& idx,
                              const std::vector<TileArgs>& targs, int64_t n, const int64_t* nsw,
                              int64_t* const* dev_EM, const BatchOptions& opt, char* work,
                              size_t work_bytes, int blocks) {
  hipStream_t stream = hs[idx[0]]->stream;
  const int nl = (int)idx.size();
  std::vector<FusedLattice> lat(nl);
  std::vector<FusedTile> tiles;
  bool any_em = false;
  // Every lattice keeps the tile shape of the plan (coarser tiles for the
  // largest lattices helped a batch made mostly of them, +1.9 % on the
  // 224-lattice grid, but unbalanced served mixes: p50 latency 1.7 -> 3.0 s).
  for (int j = 0; j < nl; ++j) {
    const int i = idx[j];
    FusedLattice& F = lat[j];
    std::memset(&F, 0, sizeof(F));
    F.ta = targs[i];
    make_flat(F.ta, true);  // the fused kernel uses the flat mapping for every lattice
    F.ta.t = (uint32_t)hs[i]->sweep;
    F.EM = dev_EM ? dev_EM[i] : nullptr;
    any_em = any_em || F.EM != nullptr;
    F.ntiles = F.ta.tiles;
    F.nsweeps = nsw ? nsw[i] : n;
  }
  // The grid deals the tile list out with a static stride.  Listing the
  // larger tiles first (two row groups per wave before one), and within a
  // size the lattices that run the most sweeps of this launch first, gives
  // every workgroup about the same work per round (longest first), and the
  // tiles of lattices that finish early in a chunk drop out of the end of
  // the list.  Results do not depend on the order.
  std::vector<int> order(nl);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
    if (lat[a].ta.RPW != lat[b].ta.RPW) return lat[a].ta.RPW > lat[b].ta.RPW;
    return lat[a].nsweeps > lat[b].nsweeps;
  });
  for (int j : order) {
    lat[j].first_tile = (int64_t)tiles.size();
    for (int64_t t = 0; t < lat[j].ntiles; ++t) tiles.push_back(FusedTile{j, (int32_t)t});
  }
  const int64_t ntiles = (int64_t)tiles.size();
  blocks = (int)std::min<int64_t>(blocks, std::max<int64_t>(ntiles, 1));
  const FusedLayout fl = fused_layout(nl, ntiles);
  if (fl.bytes > work_bytes)
    return fail(ISING_ENOMEM, "batched sweeps: work buffer of %zu bytes < %zu needed", work_bytes,
                fl.bytes);
  // the image covers the sweep counter (zero) and the tables; the partials
  // are written before they are read
  const bool async = opt.keep_image != nullptr && opt.graph_chunk == 0;
  std::vector<char> local;
  std::vector<char>& img = async ? *opt.keep_image : local;
  img.assign(fl.off_part, 0);
  std::memcpy(img.data() + fl.off_lat, lat.data(), nl * sizeof(FusedLattice));
  std::memcpy(img.data() + fl.off_tiles, tiles.data(), ntiles * sizeof(FusedTile));
  hipError_t e = hipMemcpyAsync(work, img.data(), img.size(), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return hip_fail(e, "batched sweeps: table upload");
  // a local image ends with this call: wait for its upload
  if (!async) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return hip_fail(e, "batched sweeps: table upload");

  FusedArgs f;
  f.lat = (const FusedLattice*)(work + fl.off_lat);
  f.nlat = nl;
  f.klocal = 0;
  f.tiles = (const FusedTile*)(work + fl.off_tiles);
  f.ntiles = ntiles;
  f.kbase = (const uint32_t*)(work + fl.off_k);
  f.part = (uint32_t*)(work + fl.off_part);
  uint32_t* kbase = (uint32_t*)(work + fl.off_k);

  int64_t done = 0;
  const int K = opt.graph_chunk;
  if (K > 0 && n >= 2 * (int64_t)K) {
    // capture K sweeps (+ the counter advance) once on a private stream,
    // then replay the chunk n / K times on the caller's stream
    DeviceState& D = state_for(hs[idx[0]]->device);
    std::lock_guard<std::mutex> lock(D.m);
    if (!D.capture) {
      e = hipStreamCreateWithFlags(&D.capture, hipStreamNonBlocking);
      if (e != hipSuccess) return hip_fail(e, "batched sweeps: capture stream");
    }
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    e = hipStreamBeginCapture(D.capture, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      for (int k = 0; k < K && e == hipSuccess; ++k) {
        f.klocal = k;
        e = launch_fused(D.capture, 0, f, blocks);
        if (e == hipSuccess) e = launch_fused(D.capture, 1, f, blocks);
      }
      if (e == hipSuccess) e = launch_advance(D.capture, kbase, (uint32_t)K);
      hipError_t e2 = hipStreamEndCapture(D.capture, &graph);
      if (e == hipSuccess) e = e2;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    const int64_t reps = n / K;
    for (int64_t r = 0; r < reps && e == hipSuccess; ++r) e = hipGraphLaunch(exec, stream);
    // the executable graph may be destroyed once its launches are enqueued
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return hip_fail(e, "batched sweeps: graph capture/replay");
    done = reps * K;
  }
  // remaining sweeps: direct launches at kbase + klocal; the device counter
  // moves on every 2^20 sweeps so that klocal stays small
  const int64_t kStep = int64_t(1) << 20;
  int64_t base = 0;
  for (int64_t k = 0; k < n - done; ++k) {
    if (k - base == kStep) {
      e = launch_advance(stream, kbase, (uint32_t)kStep);
      if (e != hipSuccess) return hip_fail(e, "batched sweeps: counter advance");
      base = k;
    }
    f.klocal = (int32_t)(k - base);
    e = launch_fused(stream, 0, f, blocks);
    if (e == hipSuccess) e = launch_fused(stream, 1, f, blocks);
    if (e != hipSuccess) return hip_fail(e, "batched sweeps: fused launch");
  }
  if (any_em) {
    // the last sweep: kbase + klocal = n - 1
    f.klocal = n - done > 0 ? (int32_t)(n - done - 1 - base) : -1;
    e = launch_fused_finalize(stream, f, std::min(nl, 1024));
    if (e != hipSuccess) return hip_fail(e, "batched sweeps: finalize launch");
  }
  if (async) return ISING_OK;
  e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return hip_fail(e, "batched sweeps: synchronize");
  return ISING_OK;
}

// All lattices idx (shapes in plan, in order) in the block form.
static ising_status run_blocks(ising_lattice* const* hs, const std::vector<int>& idx, int64_t n,
                               const int64_t* nsw, int64_t* const* dev_EM, const BlockPlan& plan,
                               char* work, std::vector<char>* keep_image) {
  hipStream_t stream = hs[idx[0]]->stream;
  const int nl = (int)idx.size();
  std::vector<BlockLattice> lat(nl);
  std::vector<BlockTask> tasks;
  int launches = 0, threads = 0;
  size_t lds = 0;
  bool finalize = false;
  // the longest strips first, so that none starts late
  std::vector<int> order(nl);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
    return plan.shapes[a].step_s > plan.shapes[b].step_s;
  });
  for (int j = 0; j < nl; ++j) {
    const int i = idx[j];
    lat[j] = block_lattice(hs[i], plan.shapes[j], nsw ? nsw[i] : n, plan.all_single,
                           dev_EM ? dev_EM[i] : nullptr);
    launches = std::max(launches, (int)lat[j].launches);
    threads = std::max(threads, (int)lat[j].threads);
    lds = std::max(lds, plan.shapes[j].lds);
    finalize = finalize || (lat[j].strips > 1 && lat[j].EM != nullptr);
  }
  for (int j : order)
    for (int32_t s = 0; s < lat[j].strips; ++s) tasks.push_back(BlockTask{j, s});
  const BlockLayout bl = block_layout(nl, tasks.size());
  std::vector<char> local;
  std::vector<char>& img = keep_image ? *keep_image : local;
  img.assign(bl.bytes, 0);
  std::memcpy(img.data(), lat.data(), nl * sizeof(BlockLattice));
  std::memcpy(img.data() + bl.off_tasks, tasks.data(), tasks.size() * sizeof(BlockTask));
  hipError_t e = hipMemcpyAsync(work, img.data(), img.size(), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return hip_fail(e, "batched sweeps: table upload");
  const BlockLattice* tab = (const BlockLattice*)work;
  for (int j = 0; j < launches && e == hipSuccess; ++j)
    e = launch_block_many(stream, tab, (const BlockTask*)(work + bl.off_tasks), (int)tasks.size(),
                          device_cus(hs[idx[0]]->device), threads, lds, j);
  if (e == hipSuccess && finalize) e = launch_block_finalize_many(stream, tab, nl);
  // the host image must outlive the upload: wait before it goes, unless the
  // caller keeps it
  if (e == hipSuccess && !keep_image) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return hip_fail(e, "batched sweeps: block launch");
  return ISING_OK;
}

// Which lattices take the tiled batched kernels (their tile arguments in
// targs) and which the plain path.
static void classify(ising_lattice* const* hs, int32_t count, const BatchOptions& opt,
                     std::vector<int>& tiled, std::vector<int>& other,
                     std::vector<TileArgs>& targs) {
  targs.assign(count, TileArgs{});
  for (int i = 0; i < count; ++i) {
    TileArgs ta;
    // the fused kernel indexes a plane with 32-bit word numbers: planes of
    // 2^32 words or more (L >= 741456) take the plain path
    if (tile_args(hs[i], &ta) && hs[i]->plane_words < (1ll << 32)) {
      // fine tiles balance best across the flat list; lattices with many
      // tiles take up to rpw_max row groups per wave (kTileMaxWords words of a
      // tile at most)
      const int64_t TR1 = 4 * (int64_t)ta.R;
      const int64_t tiles1 = ((hs[i]->L + TR1 - 1) / TR1) * ta.segs;
      int rpw = 1;
      for (int r = 2; r <= opt.rpw_max; r *= 2) {
        if (tiles1 < 128 * (int64_t)r || (r * TR1 + 2) * (ta.TW + 2) > kTileMaxWords) break;
        rpw = r;
      }
      ta.RPW = rpw;
      const int64_t TR = TR1 * rpw;
      ta.tiles = ((hs[i]->L + TR - 1) / TR) * ta.segs;
      targs[i] = ta;
      tiled.push_back(i);
    } else {
      other.push_back(i);
    }
  }
  // one large lattice alone runs faster on the plain path (its own tuned
  // shape, no tile table): 4096^2 1345-1366 against 1140 updates/ns fused
  if (opt.force_form < 0 && tiled.size() == 1 && hs[tiled[0]]->plane_words >= (int64_t)1 << 16) {
    other.push_back(tiled[0]);
    tiled.clear();
  }
}

// Work-buffer bytes for the tiled lattices: the larger of the two forms.
static size_t work_bytes_for(ising_lattice* const* hs, const std::vector<int>& tiled,
                             const std::vector<TileArgs>& targs,
                             size_t record = sizeof(FusedLattice)) {
  if (tiled.empty()) return 0;
  size_t ntiles = 0;
  for (int i : tiled) ntiles += (size_t)fused_tiles(hs[i]->plane_words, targs[i].RPW);
  const size_t nl = tiled.size();
  return std::max(fused_layout(nl, ntiles, record).bytes, block_layout(nl, nl).bytes);
}

// Whether every lattice that the plan cuts into strips has a copy of its own:
// strips of one launch write all of them.
static bool own_spares(ising_lattice* const* hs, const BlockPlan& plan) {
  std::vector<std::pair<uintptr_t, size_t>> at;
  for (size_t i = 0; i < plan.shapes.size(); ++i) {
    if (plan.shapes[i].strips == 1) continue;
    if (!hs[i]->spare) return false;
    at.push_back({(uintptr_t)hs[i]->spare, ising_spare_bytes(hs[i]->L)});
  }
  std::sort(at.begin(), at.end());
  for (size_t i = 1; i < at.size(); ++i)
    if (at[i - 1].first + at[i - 1].second > at[i].first) return false;
  return true;
}

static size_t work_bytes_of(ising_lattice* const* hs, int32_t count, const BatchOptions& opt,
                            size_t record) {
  std::vector<int> tiled, other;
  std::vector<TileArgs> targs;
  classify(hs, count, opt, tiled, other, targs);
  return work_bytes_for(hs, tiled, targs, record);
}

size_t batch_work_bytes(ising_lattice* const* hs, int32_t count, const BatchOptions& opt) {
  return work_bytes_of(hs, count, opt, sizeof(FusedLattice));
}

// Block tables that a batch runs without, but faster with: lattices that the
// tiles leave to the plain path (sides no multiple of 8), one after another,
// can advance together in blocks.  200 sweeps of 16 x 1002^2 12.3 -> 2.5 ms.
static size_t optional_work_bytes(ising_lattice* const* hs, int32_t count) {
  bool odd = false, sides = true;
  double sites = 0;
  for (int i = 0; i < count; ++i) {
    odd = odd || hs[i]->L % 8 != 0;
    sides = sides && hs[i]->L <= kBlockMaxL;
    sites += (double)hs[i]->L * hs[i]->L;
  }
  return count > 1 && odd && sides && sites <= kBlockMaxSites
             ? block_layout(count, count + kBlockMaxTasks).bytes
             : 0;
}

size_t batch_work_share(int64_t L) {
  const int64_t plane_words = L * words_per_row(L);
  const size_t fused = sizeof(FusedLattice) +
                       (size_t)fused_tiles(plane_words, 1) * (sizeof(FusedTile) + 64);
  const size_t packed = sizeof(BlockLattice) + sizeof(BlockTask);
  return std::max(fused, packed);
}

ising_status batch_sweeps(ising_lattice* const* hs, int32_t count, int64_t n,
                          const int64_t* nsw, int64_t* const* dev_EM, const BatchOptions& opt,
                          void* work, size_t work_bytes, int* form_out) {
  if (form_out) *form_out = -1;
  if (count == 0 || n == 0) return ISING_OK;
  const int device = hs[0]->device;
  std::vector<int> tiled, other;
  std::vector<TileArgs> targs;
  classify(hs, count, opt, tiled, other, targs);
  if (!tiled.empty()) {
    const size_t need = work_bytes_for(hs, tiled, targs);
    if (!work || need > work_bytes || ((uintptr_t)work & 255))
      return fail(ISING_ENOMEM,
                  "batched sweeps: needs a 256-byte aligned work buffer of %zu bytes (got %zu)",
                  need, work ? work_bytes : (size_t)0);
  }
  // Blocks for the whole batch, where the caller leaves the form open, every
  // lattice can take them and the model has them ahead of a launch per colour
  // step.  (Beside a lattice that cannot, the small ones ride along in its
  // launches.)  Their tables may need more than the work buffer holds: then
  // the other forms run.
  const int cus = device_cus(device);
  int kind = kBlockCompare;
  for (int i = 0; i < count; ++i)
    if (hs[i]->cut.x) kind = kBlockPhilox;
  if (opt.force_form < 0 && work && ((uintptr_t)work & 255) == 0) {
    std::vector<int> all(count);
    std::iota(all.begin(), all.end(), 0);
    std::vector<int64_t> Ls;
    bool spares = true;
    for (int i = 0; i < count; ++i) {
      Ls.push_back(hs[i]->L);
      spares = spares && (hs[i]->spare || block_fits_single(hs[i]->L));
    }
    BlockPlan plan;
    if (spares && choose_blocks(kind, Ls, n, cus, work_bytes, &plan)) {
      if (own_spares(hs, plan)) {
        if (form_out) *form_out = plan.all_single ? 1 : 0;
        return run_blocks(hs, all, n, nsw, dev_EM, plan, (char*)work, opt.keep_image);
      }
    }
  }
  // Packed: tiled lattices that fit one workgroup run all their sweeps in one
  // launch, where that is forced, or where all of them fit and it is cheaper;
  // any others advance together in the fused form (2048 lattices of 1024^2, 10
  // sweeps: 15.5 ms, one after another 84).
  BlockPlan singles;
  std::vector<int> fits;
  if (!tiled.empty()) {
    if (cus <= 0) return fail(ISING_EDEVICE, "batched sweeps: no device properties");
    std::vector<int> rest;
    std::vector<int64_t> Ls;
    for (int i : tiled) {
      (block_fits_single(hs[i]->L) ? fits : rest).push_back(i);
      Ls.push_back(hs[i]->L);
    }
    const bool packed =
        opt.force_form == 1 || (opt.force_form < 0 && rest.empty() &&
                                choose_blocks(kind, Ls, 1, cus, work_bytes, &singles));
    if (form_out) *form_out = packed ? 1 : 0;
    if (packed) {
      tiled.swap(rest);
      if (opt.force_form == 1) {
        singles = BlockPlan();
        for (int i : fits) singles.shapes.push_back(block_shape_single(kBlockPhilox, hs[i]->L));
        singles.all_single = true;
      }
    } else {
      fits.clear();
    }
  }
  for (int i : other) {
    ising_status st = enqueue_sweeps(hs[i], nsw ? nsw[i] : n, dev_EM ? dev_EM[i] : nullptr);
    if (st != ISING_OK) return st;
  }
  if (!fits.empty()) {
    ising_status st = run_blocks(hs, fits, n, nsw, dev_EM, singles, (char*)work, opt.keep_image);
    if (st != ISING_OK) return st;
  }
  if (tiled.empty()) {
    if (opt.keep_image) return ISING_OK;
    hipError_t e = hipStreamSynchronize(hs[0]->stream);
    return e == hipSuccess ? ISING_OK : hip_fail(e, "batched sweeps: synchronize");
  }
  // the fused grid walks actual tiles; size it for them
  int64_t ntiles = 0;
  for (int i : tiled) ntiles += targs[i].tiles;
  return run_fused(hs, tiled, targs, n, nsw, dev_EM, opt, (char*)work, work_bytes,
                   fused_grid(ntiles, opt.wg_per_cu, cus));
}

}  // namespace ising

using namespace ising;

extern "C" ising_status ising_batch_plan(const int64_t* Ls, int32_t count, int32_t cus,
                                         int32_t* form_out, int32_t* blocks_out,
                                         double* est_seconds_out) {
  clear_error();
  if (!Ls || count < 1 || cus < 1 || !form_out || !blocks_out)
    return fail(ISING_EINVAL, "ising_batch_plan: bad arguments");
  int64_t tiles = 0;
  double words = 0;
  for (int32_t i = 0; i < count; ++i) {
    const int64_t L = Ls[i];
    if (L < 8 || L % 8 || L > kMaxL)
      return fail(ISING_EINVAL, "ising_batch_plan: L=%lld is not a tiled size", (long long)L);
    const int64_t W = words_per_row(L);
    const int64_t R = W >= kWideMinWords ? 1 : 64 / W;
    const int64_t segs = W >= kWideMinWords ? (W + 63) / 64 : 1;
    tiles += ((L + 4 * R - 1) / (4 * R)) * segs;
    words += (double)(L * W);
  }
  BlockPlan plan;
  const bool blocks = choose_blocks(kBlockPhilox, std::vector<int64_t>(Ls, Ls + count),
                                    kBlockPlanN, cus, SIZE_MAX, &plan);
  *form_out = blocks && plan.all_single ? 1 : 0;
  *blocks_out = blocks ? (int32_t)plan.tasks
                       : fused_grid(tiles, default_batch_options().wg_per_cu, cus);
  if (est_seconds_out)
    *est_seconds_out =
        blocks ? plan.sweep_s : launch_per_step_seconds(kBlockPhilox, words, cus);
  return ISING_OK;
}

namespace ising {
ising_status check_batch(ising_t* const* hs, int32_t count, int64_t n, const char* who) {
  if (!hs || count < 0 || n < 0) return fail(ISING_EINVAL, "%s: bad arguments", who);
  for (int32_t i = 0; i < count; ++i) {
    if (!hs[i]) return fail(ISING_EINVAL, "%s: NULL handle %d", who, i);
    if (!hs[i]->beta_set) return fail(ISING_EINVAL, "%s: handle %d has no beta", who, i);
    if (hs[i]->lcg || hs[i]->pool)
      return fail(ISING_EINVAL,
                  "%s: handle %d uses the LCG or pattern-pool dynamics (plain sweeps only)", who,
                  i);
    if (hs[i]->sweep + (uint64_t)n > (1ull << 32))
      return fail(ISING_ERANGE, "%s: counter overflow on handle %d", who, i);
    if (hs[i]->stream != hs[0]->stream || hs[i]->device != hs[0]->device)
      return fail(ISING_EINVAL, "%s: handles must share one device and stream", who);
    for (int32_t j = 0; j < i; ++j)
      if (hs[j] == hs[i]) return fail(ISING_EINVAL, "%s: handle %d repeated", who, i);
  }
  return ISING_OK;
}
}  // namespace ising

// ---------------------------------------------------------------------
// The allocation-free variant (ising_multi_sweep_static): the task tables
// live in this file-scope device array instead of a caller work buffer.
// Each GPU holds its own copy of the array for the life of the process; its
// device address is looked up once per device (hipGetSymbolAddress) and
// used from then on, never the array's host-side name.  Calls on one device
// are serialised by a per-device mutex (each call waits for its stream
// before it returns), so calls from several threads of a process do not
// overlap on the array.
// ---------------------------------------------------------------------
// A batch is taken if its tables are within 4 MiB with 240 bytes per lattice.
// The record has grown beyond that, and the array with it, by as many lattices
// as fit: each has a tile and its partials too.
constexpr size_t kStaticLimit = size_t(4) << 20, kStaticRecord = 240;
static_assert(sizeof(FusedLattice) >= kStaticRecord, "kStaticRecord");
constexpr size_t kStaticWorkBytes =
    (kStaticLimit + kStaticLimit / (kStaticRecord + sizeof(FusedTile) + 64) *
                        (sizeof(FusedLattice) - kStaticRecord) + 511) & ~size_t(255);
static __device__ __align__(256) unsigned char scratch[kStaticWorkBytes];

namespace {
struct StaticScratch {
  std::mutex m;
  void* ptr = nullptr;  // device address of `scratch` on this device
};
StaticScratch& static_scratch(int device) {
  static StaticScratch s[64];
  return s[device & 63];
}
}  // namespace

extern "C" ising_status ising_multi_sweep_static(ising_t* const* hs, int32_t count, int64_t n,
                                                 int64_t* const* dev_EM) {
  clear_error();
  ising_status st = check_batch(hs, count, n, "ising_multi_sweep_static");
  if (st != ISING_OK) return st;
  if (count == 0 || n == 0) return ISING_OK;
  BatchOptions opt = default_batch_options();
  opt.graph_chunk = 0;  // no hipGraph: instantiating one allocates
  const size_t need = work_bytes_of(hs, count, opt, kStaticRecord);
  if (need > kStaticLimit)
    return fail(ISING_ENOMEM,
                "ising_multi_sweep_static: the batch needs %zu bytes of tables, more than the "
                "%zu bytes of the static scratch",
                need, kStaticLimit);
  const int device = hs[0]->device;
  if (device < 0 || device >= 64) return fail(ISING_EINVAL, "ising_multi_sweep_static: device");
  StaticScratch& S = static_scratch(device);
  std::lock_guard<std::mutex> lock(S.m);
  if (!S.ptr) {
    int current = 0;
    hipError_t e = hipGetDevice(&current);
    if (e == hipSuccess && current != device) e = hipSetDevice(device);
    void* p = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (current != device) (void)hipSetDevice(current);
    if (e != hipSuccess || !p) return hip_fail(e, "ising_multi_sweep_static: scratch address");
    S.ptr = p;
  }
  st = batch_sweeps(hs, count, n, nullptr, dev_EM, opt, S.ptr, kStaticWorkBytes, nullptr);
  if (st != ISING_OK) return st;
  for (int32_t i = 0; i < count; ++i) hs[i]->sweep += (uint64_t)n;
  return ISING_OK;
}

extern "C" ising_status ising_multi_sweep_work_bytes(ising_t* const* hs, int32_t count,
                                                     size_t* bytes) {
  clear_error();
  if (!bytes) return fail(ISING_EINVAL, "ising_multi_sweep_work_bytes: bytes is NULL");
  *bytes = 0;
  ising_status st = check_batch(hs, count, 0, "ising_multi_sweep_work_bytes");
  if (st != ISING_OK) return st;
  // every form the caller may force and every fused shape the batched
  // autotuner may install: count each tiled lattice (a lone large lattice
  // takes the plain path only when the cost model chooses) with its finest
  // tiles
  BatchOptions opt = default_batch_options();
  opt.force_form = 0;
  opt.rpw_max = 1;
  *bytes = std::max(batch_work_bytes(hs, count, opt), optional_work_bytes(hs, count));
  return ISING_OK;
}

extern "C" ising_status ising_multi_sweep(ising_t* const* hs, int32_t count, int64_t n,
                                          int64_t* const* dev_EM, void* dev_work,
                                          size_t work_bytes) {
  return ising_multi_sweep_form(hs, count, n, dev_EM, -1, -1, dev_work, work_bytes);
}

extern "C" ising_status ising_multi_sweep_form(ising_t* const* hs, int32_t count, int64_t n,
                                               int64_t* const* dev_EM, int32_t form,
                                               int32_t graph_chunk, void* dev_work,
                                               size_t work_bytes) {
  clear_error();
  ising_status st = check_batch(hs, count, n, "ising_multi_sweep");
  if (st != ISING_OK) return st;
  if (form < -1 || form > 1 || graph_chunk < -1)
    return fail(ISING_EINVAL, "ising_multi_sweep: bad form or graph chunk");
  BatchOptions opt = default_batch_options();
  opt.force_form = form;
  if (graph_chunk >= 0) opt.graph_chunk = graph_chunk;
  st = batch_sweeps(hs, count, n, nullptr, dev_EM, opt, dev_work, work_bytes, nullptr);
  if (st != ISING_OK) return st;
  for (int32_t i = 0; i < count; ++i) hs[i]->sweep += (uint64_t)n;
  return ISING_OK;
}
