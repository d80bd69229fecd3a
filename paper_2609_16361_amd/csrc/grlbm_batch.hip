// grlbm_batch.hip -- many uneven instances stepped together (C ABI lbm_batch_*).
//
// One device arena holds the populations of every instance (the same SoA, AA
// in-place layout as a single context).  A descriptor table and a tile work-list
// live in device memory: a tile is one block-width range of consecutive cells of
// one instance.  k_batch_step loops over the tile list with a fixed grid
// (persistent) or takes one tile per block (grid 0 in the tuning), and each block
// derives its instance's AA parity and whether it is active from a device-resident
// clock, so one launch advances every active instance by one step whatever its
// size, boundaries, parameters or age.  Consecutive launches on one stream order
// the steps (no grid-wide barrier is needed).  Time loops of K steps are captured
// once in a hipGraph: K step nodes per (collision, storage) group followed by a
// one-lane kernel that advances the clock (no memset nodes), and replayed; the tile
// list, descriptors and tile count can change between replays because the graph
// only holds their addresses (with one block per tile, a change of the rounded
// grid captures the graph again).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/grlbm.h"
#include "grlbm_device.hpp"
#include "grlbm_internal.h"
#include "grlbm_pair.hpp"
#include "grlbm_tube.hpp"

namespace grlbm {

struct BatchInst {
  Coll c;
  Grid g;
  int64_t off;      // element offset of the instance's slot 0 in the arena
  int64_t t_start;  // clock value at which the instance was at its step 0
  int64_t t_end;    // clock value at which it has completed all its steps
  double inv_px;    // 1/px and 1/ny for the element-index decomposition
  double inv_ny;
  int32_t cells;    // px * ny * nz: the elements the instance's rows span
  int32_t pad_;
  TubeShape tube;   // windows of k_batch_tube, or
  PairTiles pair;   // tiles of k_batch_pair, where the instance makes several steps a pass
};

// A tile is `blockDim.x` consecutive element indices of one instance (it may span
// several x-rows; lanes on a row's padding have no cell).
struct BatchTile {
  int32_t inst;
  int32_t tile;  // tile index within the instance: cells [tile * blockDim.x, ...)
};

// A run of a tile list.
struct TileRun {
  int32_t start;
  int32_t count;
};

// q = n / d and r = n % d for 0 <= n < 2^31: the FP64 product is within one of the
// quotient, one correction step makes it exact.
__device__ __forceinline__ int div_exact(int n, int d, double inv_d, int& r) {
  int q = (int)((double)n * inv_d);
  r = n - q * d;
  if (r < 0) {
    --q;
    r += d;
  } else if (r >= d) {
    ++q;
    r -= d;
  }
  return q;
}

template <int COLL, typename T, bool NT>
__global__ void __launch_bounds__(1024) k_batch_step(T* __restrict__ arena, const BatchInst* __restrict__ insts,
                                                      const BatchTile* __restrict__ tiles,
                                                      const TileRun* __restrict__ run,
                                                      const int64_t* __restrict__ clock, int32_t j) {
  extern __shared__ float xs[];  // x slots of an odd-step tile (tile_update_odd)
  const int32_t nt = run->count;
  const int64_t t = *clock + j;
  tiles += run->start;
  for (int32_t tile = blockIdx.x; tile < nt; tile += gridDim.x) {
    const BatchTile bt = tiles[tile];
    const BatchInst* I = insts + bt.inst;
    const int64_t ts = I->t_start;
    if (t < ts || t >= I->t_end) continue;  // the same for the whole block
    const int n0 = bt.tile * (int)blockDim.x;
    const int n = n0 + (int)threadIdx.x;
    bool act = n < I->cells;
    const Grid g = I->g;
    int x = 0, y = 0, z = 0;
    if (act) {
      const int row = div_exact(n, g.px, I->inv_px, x);
      z = div_exact(row, g.ny, I->inv_ny, y);
      act = x < g.nx;  // the row's padding holds no cell
    }
    const Coll c = I->c;
    T* F = arena + I->off;
    // the same arithmetic as a single context uses for this instance, so the
    // results are bitwise the same.  Every instance takes the zero-gradient form
    // of the update: on a periodic axis its face flags are false and it reads and
    // writes exactly what the periodic form does.  A kernel holding both forms
    // compiled to 113-128 registers (94-99 with one) and ran FP16 batches of
    // periodic cubes at 21 GLUP/s against 33 with the single form.
    const bool odd = ((t - ts) & 1) != 0;
    const uint32_t skey = step_key(t - ts);  // the instance's own step index
    if (odd) {
      // every lane takes part (barriers inside).  With the nontemporal hint, the y
      // and z slots are loaded without it: on the batch of 64 Becker tubes (4 x 4
      // cells across, so rows and planes are fractions of a line) 62.35 against
      // 58.09 solves/s at the fastest launch shape, 62.00 with the y slots alone;
      // dropping it on the y and z stores as well gained nothing.
      tile_update_odd<COLL, T, true, false, NT, true, false, NT ? 2 : 0>(F, g, c, n0, act, x, y, z, xs, nullptr,
                                                                         skey);
    } else if (act) {
      cell_update<false, COLL, T, true, false, NT>(F, g, c, x, y, z, nullptr, skey);
    }
  }
}

// The tile of this block: neighbouring tiles, which share halo lines, on one XCD (blocks
// are dealt to the 8 XCDs in turn).  -1: none.
__device__ __forceinline__ int32_t xcd_tile(int32_t count) {
  const int32_t per = (count + 7) / 8, i = (int32_t)(blockIdx.x / 8);
  const int32_t tile = (int32_t)(blockIdx.x % 8) * per + i;
  return i < per && tile < count ? tile : -1;
}

// An odd and the following even step (steps j and j + 1 after the clock) of the FP32
// instances that step in pairs, one tile per block, from one arena to the other at the
// same offsets.  The host lists only instances at even parity and with all the steps of
// the run ahead of them; those that have finished since are skipped.  Every instance
// takes the zero-gradient form, as in k_batch_step.  On a serving mix of 24 requests the
// FP32 vortices (10 of 32^3-55^3) and tubes took 63 us per step in single steps; the
// vortices now take 33 and the tubes 9 (k_batch_tube).
template <int COLL>
__global__ void __launch_bounds__(kPairThreads) k_batch_pair(const char* __restrict__ from, char* __restrict__ to,
                                                              const BatchInst* __restrict__ insts,
                                                              const BatchTile* __restrict__ tiles,
                                                              const TileRun* __restrict__ run,
                                                              const int64_t* __restrict__ clock, int32_t j) {
  extern __shared__ float xs[];
  const int32_t i = xcd_tile(run->count);
  if (i < 0) return;
  const BatchTile bt = tiles[run->start + i];
  const BatchInst* I = insts + bt.inst;
  if (*clock + j >= I->t_end) return;
  const Grid g = I->g;
  const Coll c = I->c;
  const PairTiles pt = I->pair;
  const int nxy = pt.ntx * pt.nty;
  const int seg = bt.tile / nxy;
  pair_update<COLL, true, false>(reinterpret_cast<const float*>(from) + I->off, reinterpret_cast<float*>(to) + I->off,
                                 g, c, pt, seg, bt.tile - seg * nxy, xs);
}

// `steps` (even) steps from step j after the clock on of the instances that are tubes,
// one window per block, from one arena to the other.  The batch of 64 Becker tubes
// (4.5 M cells, FP32) took 237 us per step in single steps and takes 85 now; the FP16
// tubes of the serving mix 17 and 10.
template <int COLL, typename T, int L>
__global__ void __launch_bounds__(L, 4) k_batch_tube(const char* __restrict__ from, char* __restrict__ to,
                                                      const BatchInst* __restrict__ insts,
                                                      const BatchTile* __restrict__ tiles,
                                                      const TileRun* __restrict__ run,
                                                      const int64_t* __restrict__ clock, int32_t j, int32_t steps) {
  extern __shared__ float xs[];
  const int32_t i = xcd_tile(run->count);
  if (i < 0) return;
  const BatchTile bt = tiles[run->start + i];
  const BatchInst* I = insts + bt.inst;
  const int64_t t = *clock + j;
  if (t >= I->t_end) return;
  const Grid g = I->g;
  const Coll c = I->c;
  const TubeShape sh = I->tube;
  tube_update<COLL, T, L>(reinterpret_cast<const T*>(from) + I->off, reinterpret_cast<T*>(to) + I->off, g, c,
                          bt.tile * sh.inner, sh.width, sh.inner, steps, t - I->t_start, xs);
}

__global__ void k_batch_advance(int64_t* clock, int32_t n) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *clock += n;
}

// A run of cells [c0, c1) of one instance for the divergence check: element offset
// of the instance's slot 0 in the arena, elements between its slot arrays, storage,
// and the index of the instance's flag.
struct CheckItem {
  int64_t off;
  int64_t S;
  int32_t c0, c1;
  int32_t f16;
  int32_t flag;
  int32_t nx, px;  // row length and pitch: elements with (e mod px) >= nx are padding
};
constexpr int32_t kCheckRun = 16384;   // cells per item
constexpr int32_t kCheckBlocks = 16;   // blocks per item (256 lanes, 4 cells each)

// flags[item.flag] = 1 when the rest population (slot 0) of some field holds a
// non-finite value in the item's cells (exponent bits all ones: an infinity or a
// NaN, FP32 or FP16).  Slot 0 of field k after a step is a sum over all of the
// cell's field-k populations before it (Q_k / 4 in the regularized update, f_0 +
// omega (f_0^eq - f_0) with f_0^eq = Q_k / 4 in BGK), so a non-finite population of
// any field shows up there one step after it appears.  blockIdx.y picks the item;
// its kCheckBlocks blocks stride over the run.  Reads 5 of the 35 arrays.
__global__ void __launch_bounds__(256) k_batch_nonfinite(const char* __restrict__ arena,
                                                          const CheckItem* __restrict__ items,
                                                          int32_t* __restrict__ flags) {
  const CheckItem it = items[blockIdx.y];
  bool bad = false;
  for (int32_t c = it.c0 + (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); c < it.c1;
       c += (int32_t)(gridDim.x * blockDim.x)) {
    if (c % it.px >= it.nx) continue;
#pragma unroll
    for (int k = 0; k < kFields; ++k) {
      const int64_t e = it.off + (int64_t)(7 * k) * it.S + c;
      if (it.f16) {
        bad |= (reinterpret_cast<const uint16_t*>(arena)[e] & 0x7c00u) == 0x7c00u;
      } else {
        bad |= (reinterpret_cast<const uint32_t*>(arena)[e] & 0x7f800000u) == 0x7f800000u;
      }
    }
  }
  if (bad) flags[it.flag] = 1;  // every writer stores the same value
}

}  // namespace grlbm

using grlbm::BatchInst;
using grlbm::BatchTile;
using grlbm::TileRun;
using grlbm::fail;

namespace {

constexpr int kGroups = 4;  // (collision, storage) pairs
constexpr size_t kSpareArena = size_t(4) << 30;  // most of the arena that has a second one ...
constexpr size_t kSpareFirst = size_t(64) << 20;  // ... and what it starts with

int group_of(const lbm_params* p) { return p->collision * 2 + (p->storage == LBM_STORE_F16 ? 1 : 0); }

// The runs of a group's tile lists: the tiles of single steps, ordered by how their
// instance steps in a fast run (singly, in pairs, as a tube), and the tiles of pairs and
// the windows of tubes.
enum { kAll, kSingle, kPaired, kPairTiles, kWindows, kRuns };

struct HostInst {
  bool live = false;
  lbm_params p{};
  BatchInst d{};
  size_t bytes = 0;
  int group = 0;
  int pair_cus = 0;  // the share of the card that d.pair was chosen for
  int how = kSingle; // its steps in fast runs: kSingle, kPaired or kWindows
};

}  // namespace

struct lbm_batch {
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int num_cus = 256;
  char* arena = nullptr;
  size_t arena_bytes = 0;
  std::map<size_t, size_t> free_list;  // offset -> bytes
  int32_t max_inst = 0;
  int32_t max_tiles = 0;
  BatchInst* d_insts = nullptr;
  BatchTile* d_tiles = nullptr;      // kGroups segments of max_tiles: tiles of single steps
  BatchTile* d_multi = nullptr;      // the same for pair tiles and tube windows, from the
                                     // first instance on that has some
  TileRun* d_runs = nullptr;         // kGroups times kRuns
  int64_t* d_clock = nullptr;
  grlbm::CheckItem* d_check = nullptr;  // items of the divergence check (grown on demand)
  size_t check_cap = 0;
  int32_t* d_flags = nullptr;           // one flag per live instance (max_inst)
  unsigned* d_scales = nullptr;         // five words for the FP16 scales
  std::vector<HostInst> insts;
  int64_t clock = 0;
  int32_t graph_steps = 16;
  lbm_batch_tuning tune{};
  bool dirty = true;
  bool odd = false;  // the instances that make several steps per pass are at an odd step
  TileRun runs[kGroups][kRuns] = {};
  // the second arena, for the instances that lie in its reach, and the tube passes of
  // each group: lanes (0: no tubes) and most steps per launch
  grlbm::Spare spare;
  int32_t tube_lanes[kGroups] = {}, tube_steps[kGroups] = {};
  bool single_steps = false;  // lbm_batch_autotune times the single-step kernels
  bool captured = false;      // a run has been captured by the caller
  bool lost = false;          // a launch failed inside a run
  int64_t fast_steps = 0;     // steps of fast runs
  int64_t launches = 0;       // of step kernels, here or into a graph
  // captured graphs of graph_steps steps, all single and fast, and what they hold
  struct Graph {
    hipGraphExec_t exec = nullptr;
    const void* to = nullptr;  // the second arena that a fast one names
    int32_t plan[kGroups * (kRuns + 2)] = {};
  } graphs[2];
};

namespace {

int64_t inst_tiles(const lbm_params* p, int block) {
  const int64_t n = grlbm::row_pitch(p) * p->ny * p->nz;
  return (n + block - 1) / block;
}

// How an instance that the second arena reaches steps in fast runs.
int fast_way(const lbm_params& p, const grlbm::Grid& g) {
  if ((int64_t)p.ny * p.nz <= grlbm::kTubeCross) return kWindows;
  return p.storage != LBM_STORE_F16 && g.S < (int64_t(1) << 29) && grlbm::pair_worth(g) ? kPaired : kSingle;
}

// The second arena that the instances need which step several times per pass (0: none
// does): up to the end of the last one in the first arena, and a power of two, so that it
// is seldom taken anew.  (A driver that clears freed memory makes a process wait that
// frees gigabytes for nothing: a batch of 20 MB in an arena of 4 GiB took 112 ms to
// destroy with a second arena of 4 GiB, 0.4 without.)
size_t spare_need(const lbm_batch* b) {
  size_t end = 0;
  for (const HostInst& h : b->insts)
    if (h.live && fast_way(h.p, h.d.g) != kSingle)
      end = std::max(end, (size_t)h.d.off * (h.p.storage == LBM_STORE_F16 ? 2 : 4) + h.bytes);
  if (end == 0) return 0;
  size_t need = kSpareFirst;
  while (need < end && need < kSpareArena) need *= 2;
  return std::min(need, b->arena_bytes);
}

// The second arena, of at least `bytes`, and the lists of its tiles; without either the
// steps are single.
void prepare_fast(lbm_batch* b, size_t bytes) {
  grlbm::take_spare(b->spare, bytes);
  grlbm::grow_spare(b->spare, bytes);
  int dev = -1;
  {
    const std::unique_lock<std::mutex> use = b->spare.hold();
    if (b->d_multi || !b->spare.buf || hipGetDevice(&dev) != hipSuccess || dev != b->spare.device) return;
  }
  const grlbm::RelaxedCapture relaxed;
  if (hipMalloc((void**)&b->d_multi, sizeof(BatchTile) * (size_t)b->max_tiles * kGroups) != hipSuccess) {
    (void)hipGetLastError();
    b->d_multi = nullptr;
  }
}

// Chooses how each live instance makes its steps in fast runs.  Tubes and FP32 grids do
// several per pass if they lie in reach of the second arena and at the same parity as
// most of them (by cells): a fast run starts with all of them at an even step.
void plan_passes(lbm_batch* b) {
  for (HostInst& h : b->insts) h.how = kSingle;
  for (int g = 0; g < kGroups; ++g) b->tube_lanes[g] = 0;
  b->odd = false;
  if (!b->spare.buf || !b->d_multi) return;
  const auto way = [&](const HostInst& h) {
    const bool f16 = h.p.storage == LBM_STORE_F16;
    if (!h.live || h.d.t_end <= b->clock || (size_t)h.d.off * (f16 ? 2 : 4) + h.bytes > b->spare.bytes)
      return (int)kSingle;
    return fast_way(h.p, h.d.g);
  };
  const auto cells_of = [](const HostInst& h) { return (double)h.p.nx * h.p.ny * h.p.nz; };
  const auto odd_now = [&](const HostInst& h) { return ((b->clock - h.d.t_start) & 1) != 0; };
  double at[2] = {};
  for (const HostInst& h : b->insts)
    if (way(h) != kSingle) at[odd_now(h)] += cells_of(h);
  b->odd = at[1] > at[0];
  double pair_cells[kGroups] = {}, tube_cells[kGroups] = {};
  for (HostInst& h : b->insts) {
    const int how = way(h);
    if (how == kSingle || odd_now(h) != b->odd) continue;
    h.how = how;
    (how == kWindows ? tube_cells : pair_cells)[h.group] += cells_of(h);
  }
  for (int g = 0; g < kGroups; ++g) {
    // the tubes of a group share a launch, hence its lanes and steps: the cheapest for
    // their windows together.  Against them stand single steps, about 4 us + cells /
    // 18000 us (FP32) or / 24000 us (FP16) in a batch.
    const bool f16 = (g & 1) != 0;
    double best = 4.0 + tube_cells[g] / (f16 ? 24000.0 : 18000.0);
    for (int lanes : {256, 512})
      for (int steps = 2; steps <= grlbm::kTubeSteps; steps += 2) {
        int64_t blocks = 0;
        double lines = 0.0;
        for (const HostInst& h : b->insts) {
          if (h.how != kWindows || h.group != g) continue;
          const lbm_params& p = h.p;
          const int64_t cross = (int64_t)p.ny * p.nz;
          const int width = (int)(lanes / cross), inner = width - 2 * steps;
          if (inner < 2) blocks = INT32_MAX;
          if (blocks >= INT32_MAX) break;
          const int64_t windows = ((int64_t)p.nx + inner - 1) / inner;
          blocks += windows;
          lines += (double)windows * grlbm::tube_lines(cross, width, f16);
        }
        if (blocks == 0 || blocks >= INT32_MAX) continue;
        const double cost = grlbm::tube_price({lanes, 0, 0, steps, 0}, lines / (double)blocks, blocks, f16, b->num_cus);
        if (cost < best) {
          best = cost;
          b->tube_lanes[g] = lanes;
          b->tube_steps[g] = steps;
        }
      }
    for (HostInst& h : b->insts) {
      if (h.how != kWindows || h.group != g) continue;
      if (!b->tube_lanes[g]) {
        h.how = kSingle;
        continue;
      }
      const int width = b->tube_lanes[g] / (h.p.ny * h.p.nz);
      h.d.tube = {b->tube_lanes[g], width, width - 2 * b->tube_steps[g], b->tube_steps[g], 0};
    }
  }
  for (HostInst& h : b->insts) {
    if (h.how != kPaired) continue;
    // tiles for the instance's share of the card, rounded down (the shares must not add up
    // to more than the card, or its last tiles run alone) to three binary digits, so that
    // small changes of the batch keep them
    int cus = std::max(1, (int)(b->num_cus * (cells_of(h) / pair_cells[h.group])));
    for (int drop = 1; cus / drop >= 8; drop *= 2) cus = cus / drop * drop;
    if (h.pair_cus != cus) {
      h.d.pair = grlbm::pair_tiles(h.d.g, cus, true);
      h.pair_cus = cus;
    }
  }
}

lbm_status upload(lbm_batch* b) {
  if (!b->dirty) return LBM_OK;
  plan_passes(b);
  std::vector<BatchTile> tiles[kGroups], multi[kGroups];
  for (int g = 0; g < kGroups; ++g) {
    TileRun* runs = b->runs[g];
    for (int pass : {kSingle, kPaired, kWindows}) {
      const int32_t t0 = (int32_t)tiles[g].size(), m0 = (int32_t)multi[g].size();
      for (int32_t id = 0; id < (int32_t)b->insts.size(); ++id) {
        const HostInst& h = b->insts[id];
        // an instance that has completed its steps keeps its slot but no tiles
        if (!h.live || h.group != g || h.how != pass || h.d.t_end <= b->clock) continue;
        const int64_t n = inst_tiles(&h.p, b->tune.block);
        for (int64_t t = 0; t < n; ++t) tiles[g].push_back({id, (int32_t)t});
        int64_t m = 0;
        if (pass == kPaired) m = (int64_t)h.d.pair.ntx * h.d.pair.nty * h.d.pair.nseg;
        if (pass == kWindows) m = ((int64_t)h.p.nx + h.d.tube.inner - 1) / h.d.tube.inner;
        for (int64_t t = 0; t < m; ++t) multi[g].push_back({id, (int32_t)t});
      }
      const int32_t tn = (int32_t)tiles[g].size() - t0, mn = (int32_t)multi[g].size() - m0;
      if (pass == kSingle) runs[kSingle] = {t0, tn};
      if (pass == kPaired) runs[kPaired] = {t0, tn};
      if (pass == kPaired) runs[kPairTiles] = {m0, mn};
      if (pass == kWindows) runs[kWindows] = {m0, mn};
    }
    runs[kAll] = {0, (int32_t)tiles[g].size()};
    if ((int64_t)tiles[g].size() > b->max_tiles)
      return fail(LBM_ENOMEM, "tile list of %zu exceeds the batch capacity %d", tiles[g].size(), b->max_tiles);
    if ((int64_t)multi[g].size() > b->max_tiles) {  // no room for their tiles: single steps
      runs[kSingle] = runs[kAll];
      runs[kPaired] = runs[kPairTiles] = runs[kWindows] = {0, 0};
      multi[g].clear();
    }
  }
  std::vector<BatchInst> desc(b->insts.size());
  for (size_t i = 0; i < b->insts.size(); ++i) desc[i] = b->insts[i].d;
  if (!desc.empty())
    HIP_TRY(hipMemcpyAsync(b->d_insts, desc.data(), desc.size() * sizeof(BatchInst), hipMemcpyHostToDevice,
                           b->stream));
  for (int g = 0; g < kGroups; ++g) {
    if (!tiles[g].empty())
      HIP_TRY(hipMemcpyAsync(b->d_tiles + (size_t)g * b->max_tiles, tiles[g].data(),
                             tiles[g].size() * sizeof(BatchTile), hipMemcpyHostToDevice, b->stream));
    if (!multi[g].empty())
      HIP_TRY(hipMemcpyAsync(b->d_multi + (size_t)g * b->max_tiles, multi[g].data(),
                             multi[g].size() * sizeof(BatchTile), hipMemcpyHostToDevice, b->stream));
  }
  HIP_TRY(hipMemcpyAsync(b->d_runs, b->runs, sizeof(b->runs), hipMemcpyHostToDevice, b->stream));
  // the host arrays above must outlive the copies
  HIP_TRY(hipStreamSynchronize(b->stream));
  b->dirty = false;
  return LBM_OK;
}

unsigned active_groups(const lbm_batch* b) {
  unsigned m = 0;
  for (int g = 0; g < kGroups; ++g)
    if (b->runs[g][kAll].count > 0) m |= 1u << g;
  return m;
}

// Blocks launched for group g.  A fixed grid loops over the tiles (persistent); grid
// 0 gives every tile its own block, rounded up to a multiple of kGridQuantum so
// that small changes of the tile count keep a captured graph (the extra blocks
// find no tile and exit).
constexpr int32_t kGridQuantum = 256;

int32_t rounded(int32_t tiles) { return (std::max<int32_t>(tiles, 1) + kGridQuantum - 1) / kGridQuantum * kGridQuantum; }

int32_t launch_grid(const lbm_batch* b, int g, int run) {
  return b->tune.grid > 0 ? b->tune.grid : rounded(b->runs[g][run].count);
}

// Calls fn with a kernel-selecting tag of group g: its collision and storage type.
template <typename F>
hipError_t for_group(int g, F fn) {
  switch (g) {
    case 0: return fn(std::integral_constant<int, 0>(), float());
    case 1: return fn(std::integral_constant<int, 0>(), _Float16());
    case 2: return fn(std::integral_constant<int, 1>(), float());
    default: return fn(std::integral_constant<int, 1>(), _Float16());
  }
}

// The last launch's error.
hipError_t launched(lbm_batch* b) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) ++b->launches;
  return e;
}

// One step of the tiles of a run of group g, in the arena.
hipError_t launch_single(lbm_batch* b, int g, int run, int32_t j) {
  return for_group(g, [&](auto coll, auto zero) {
    using T = decltype(zero);
    constexpr int C = decltype(coll)::value;
    int lds = b->tune.blocks_per_cu > 0 ? (int)(grlbm::kLdsPerCU / (b->tune.blocks_per_cu + 1)) + 256 : 0;
    if (lds > 65536) lds = 65536;
    const int need = 15 * (int)sizeof(float) * b->tune.block;  // odd-step x slots of one tile
    if (lds < need) lds = need;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)launch_grid(b, g, run)), dim3((unsigned)b->tune.block), lds, b->stream,
                         reinterpret_cast<T*>(b->arena), b->d_insts, b->d_tiles + (size_t)g * b->max_tiles,
                         b->d_runs + g * kRuns + run, b->d_clock, j);
      return launched(b);
    };
    return b->tune.nontemporal ? go(grlbm::k_batch_step<C, T, true>) : go(grlbm::k_batch_step<C, T, false>);
  });
}

hipError_t launch_pairs(lbm_batch* b, int g, const void* from, void* to, int32_t j) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)rounded(b->runs[g][kPairTiles].count)), dim3(grlbm::kPairThreads),
                       grlbm::kPairLds, b->stream, (const char*)from, (char*)to, b->d_insts,
                       b->d_multi + (size_t)g * b->max_tiles, b->d_runs + g * kRuns + kPairTiles, b->d_clock, j);
    return launched(b);
  };
  return g < 2 ? go(grlbm::k_batch_pair<0>) : go(grlbm::k_batch_pair<1>);
}

hipError_t launch_tubes(lbm_batch* b, int g, const void* from, void* to, int32_t j, int32_t steps) {
  return for_group(g, [&](auto coll, auto zero) {
    using T = decltype(zero);
    constexpr int C = decltype(coll)::value;
    const int32_t count = b->runs[g][kWindows].count;
    const grlbm::TubeShape sh{b->tube_lanes[g], 0, 0, 0, 0};
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)rounded(count)), dim3(sh.lanes),
                         grlbm::tube_lds(sh, rounded(count), b->num_cus), b->stream, (const char*)from, (char*)to,
                         b->d_insts, b->d_multi + (size_t)g * b->max_tiles, b->d_runs + g * kRuns + kWindows,
                         b->d_clock, j, steps);
      return launched(b);
    };
    return sh.lanes == 256 ? go(grlbm::k_batch_tube<C, T, 256>) : go(grlbm::k_batch_tube<C, T, 512>);
  });
}

hipError_t launch_advance(lbm_batch* b, int32_t n) {
  hipLaunchKernelGGL(grlbm::k_batch_advance, dim3(1), dim3(64), 0, b->stream, b->d_clock, n);
  return hipGetLastError();
}

// Enqueue n single steps of every instance.
lbm_status enqueue_steps(lbm_batch* b, int32_t n) {
  for (int32_t j = 0; j < n; ++j)
    for (int g = 0; g < kGroups; ++g)
      if (b->runs[g][kAll].count > 0) HIP_TRY(launch_single(b, g, kAll, j));
  HIP_TRY(launch_advance(b, n));
  return LBM_OK;
}

// Enqueue n (even, >= fast_least) steps, several per pass where the instances can: tubes in an
// even number of launches, the rest of FP32 as one step, pairs and the odd steps left.
// The passes of each are even in number, so that all states end in the arena; where one
// cannot be launched, states are left between the two arenas.
lbm_status enqueue_fast(lbm_batch* b, int32_t n) {
  for (int g = 0; g < kGroups; ++g) {
    const TileRun* runs = b->runs[g];
    void *from = b->arena, *to = b->spare.buf;
    if (runs[kWindows].count > 0) {
      const int32_t most = b->tube_steps[g];
      const int32_t m = most > 2 ? n : n / 4 * 4;
      int32_t left = m / 2;  // in steps of two, dealt evenly
      for (int32_t i = (m + 2 * most - 1) / (2 * most) * 2; i > 0; --i) {
        const int32_t two = left / i;
        HIP_TRY(launch_tubes(b, g, from, to, m - 2 * left, 2 * two));
        left -= two;
        std::swap(from, to);
      }
      if (m < n) {  // two steps a launch and two left: once there, and copied back
        HIP_TRY(launch_tubes(b, g, from, to, m, 2));
        HIP_TRY(launch_tubes(b, g, to, from, m, 0));
      }
    }
    if (runs[kPairTiles].count > 0) {
      int32_t j = 0;
      HIP_TRY(launch_single(b, g, kPaired, j++));
      for (; j + 4 < n; j += 4) {
        HIP_TRY(launch_pairs(b, g, from, to, j));
        HIP_TRY(launch_pairs(b, g, to, from, j + 2));
      }
      for (; j < n; ++j) HIP_TRY(launch_single(b, g, kPaired, j));
    }
    if (runs[kSingle].count > 0)
      for (int32_t j = 0; j < n; ++j) HIP_TRY(launch_single(b, g, kSingle, j));
  }
  HIP_TRY(launch_advance(b, n));
  return LBM_OK;
}

void drop_graphs(lbm_batch* b) {
  for (auto& gr : b->graphs) {
    if (gr.exec) (void)hipGraphExecDestroy(gr.exec);
    gr.exec = nullptr;
  }
}

// The graph of graph_steps steps, captured anew if the launches it holds have changed.
lbm_status ready_graph(lbm_batch* b, bool fast) {
  lbm_batch::Graph& gr = b->graphs[fast ? 1 : 0];
  int32_t plan[kGroups * (kRuns + 2)] = {};
  for (int g = 0, i = 0; g < kGroups; ++g) {
    for (int r = 0; r < kRuns; ++r) {
      const bool used = b->runs[g][r].count > 0 && (fast ? r != kAll : r == kAll);
      plan[i++] = !used ? 0 : (r == kPairTiles || r == kWindows ? rounded(b->runs[g][r].count) : launch_grid(b, g, r));
    }
    if (fast) {
      plan[i] = b->tube_lanes[g];
      plan[i + 1] = b->tube_steps[g];
    }
    i += 2;
  }
  if (gr.exec && std::memcmp(plan, gr.plan, sizeof plan) == 0) return LBM_OK;
  if (gr.exec) (void)hipGraphExecDestroy(gr.exec);
  gr.exec = nullptr;
  hipGraph_t g = nullptr;
  HIP_TRY(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
  lbm_status st = fast ? enqueue_fast(b, b->graph_steps) : enqueue_steps(b, b->graph_steps);
  hipError_t e = hipStreamEndCapture(b->stream, &g);
  if (st != LBM_OK) {
    if (g) (void)hipGraphDestroy(g);
    return st;
  }
  if (e != hipSuccess) return fail(LBM_EDEVICE, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
  e = hipGraphInstantiate(&gr.exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) {
    gr.exec = nullptr;
    return fail(LBM_EDEVICE, "hipGraphInstantiate failed: %s", hipGetErrorString(e));
  }
  gr.to = fast ? b->spare.buf : nullptr;
  std::memcpy(gr.plan, plan, sizeof plan);
  return LBM_OK;
}

// Steps from the current clock on for which every instance that makes several per pass
// still has steps to make (finished ones are skipped on the device): up to the first
// that finishes.
int64_t fast_reach(const lbm_batch* b, int64_t clock) {
  bool any = false;
  for (int g = 0; g < kGroups; ++g) any |= b->runs[g][kPairTiles].count > 0 || b->runs[g][kWindows].count > 0;
  if (!any || !b->spare.buf || b->single_steps || b->captured) return 0;
  int64_t reach = INT64_MAX;
  for (const HostInst& h : b->insts)
    if (h.live && h.how != kSingle && h.d.t_end > clock) reach = std::min(reach, h.d.t_end - clock);
  return reach;
}

// The fewest steps of a fast run.  With pairs, which leave two of its steps single and
// split them from the other instances' launches, fewer than eight gain nothing (batches of
// vortices alone 0.99 of the time of single steps at 6 steps, 0.78 at 8; with tubes 1.05
// and 0.82); tubes gain from four (0.6-0.7).
int64_t fast_least(const lbm_batch* b) {
  for (int g = 0; g < kGroups; ++g)
    if (b->runs[g][kPairTiles].count > 0) return 8;
  return 4;
}

lbm_status check_kept(const lbm_batch* b) {
  return b->lost ? fail(LBM_ESTATE, "the batch's states were lost when a launch failed") : LBM_OK;
}

lbm_status run_steps(lbm_batch* b, int64_t n) {
  lbm_status st = check_kept(b);
  if (st != LBM_OK) return st;
  if ((b->dirty || !b->spare.asked) && !grlbm::capturing(b->stream))
    if (const size_t need = spare_need(b)) {
      const bool asked = b->spare.asked;
      prepare_fast(b, need);
      if (b->spare.asked != asked) b->dirty = true;  // lists with fast steps
    }
  // the second arena stays where it is until everything that uses it is enqueued; where
  // it has been given up or replaced the lists and the graph that name it are made anew
  const std::unique_lock<std::mutex> use = b->spare.hold();
  if (b->graphs[1].exec && b->graphs[1].to != b->spare.buf) {
    (void)hipGraphExecDestroy(b->graphs[1].exec);
    b->graphs[1].exec = nullptr;
    b->dirty = true;
  }
  // Under the caller's capture the steps are single: a launch kept in the caller's graph
  // would name the second arena after it has been given up, and would step past the end
  // of an instance when it is replayed.  Replays move the device's clock and not the
  // host's, which fast runs rely on, so the steps stay single from then on.
  if (n > 0 && grlbm::capturing(b->stream)) b->captured = true;
  st = upload(b);
  if (st != LBM_OK) return st;
  if (active_groups(b) == 0 || n == 0) {
    // nothing to update: the clock still moves so instance windows stay consistent
    if (n > 0) HIP_TRY(launch_advance(b, (int32_t)n));
    b->clock += n;
    return LBM_OK;
  }
  // Fast steps while no instance finishes within them.  Fast runs start at an even step of
  // the instances that make several steps per pass and are even; after a run of odd
  // length the next one that is long enough makes a single step first.  (To list the
  // instances anew after each odd run takes an upload and a wait for the stream: runs of
  // one step of 14 instances 63 us instead of 39, of three 45 us a step instead of 37.)
  const int64_t least = fast_least(b);
  const bool align = b->odd && n > least && fast_reach(b, b->clock + 1) >= least;
  for (int64_t left = n, m = 0; left > 0; left -= m) {
    const int64_t reach = b->odd ? 0 : fast_reach(b, b->clock);
    const bool one = align && left == n;
    const bool graph = !one && b->graph_steps > 1 && left >= b->graph_steps;
    m = one ? 1 : (graph ? b->graph_steps : std::min<int64_t>(left, 1 << 20));
    const bool fast = reach >= least && m >= least && (graph ? m % 2 == 0 && m <= reach : true);
    if (graph) {
      st = ready_graph(b, fast);
      if (st != LBM_OK) return st;
      HIP_TRY(hipGraphLaunch(b->graphs[fast ? 1 : 0].exec, b->stream));
    } else {
      if (fast) m = std::min(m, reach) / 2 * 2;
      const int64_t before = b->launches;
      st = fast ? enqueue_fast(b, (int32_t)m) : enqueue_steps(b, (int32_t)m);
      if (st != LBM_OK) {
        b->lost = b->launches != before;  // some steps are on their way, the clock is not
        return st;
      }
    }
    // chunk by chunk, as the device's clock, so that they agree where a later chunk fails
    b->clock += m;
    if (fast) b->fast_steps += m;
    if (m % 2 != 0) b->odd = !b->odd;
    // instances finished inside this run drop out of the tile list next time
    for (const HostInst& h : b->insts)
      if (h.live && h.d.t_end <= b->clock && h.d.t_end > b->clock - m) b->dirty = true;
  }
  return LBM_OK;
}

bool arena_alloc(lbm_batch* b, size_t bytes, size_t* off) {
  for (auto it = b->free_list.begin(); it != b->free_list.end(); ++it) {
    if (it->second >= bytes) {
      *off = it->first;
      const size_t rest = it->second - bytes;
      const size_t at = it->first + bytes;
      b->free_list.erase(it);
      if (rest) b->free_list[at] = rest;
      return true;
    }
  }
  return false;
}

void arena_free(lbm_batch* b, size_t off, size_t bytes) {
  auto it = b->free_list.emplace(off, bytes).first;
  auto nx = std::next(it);
  if (nx != b->free_list.end() && it->first + it->second == nx->first) {
    it->second += nx->second;
    b->free_list.erase(nx);
  }
  if (it != b->free_list.begin()) {
    auto pv = std::prev(it);
    if (pv->first + pv->second == it->first) {
      pv->second += it->second;
      b->free_list.erase(it);
    }
  }
}

lbm_status check_id(lbm_batch* b, int32_t id) {
  if (!b) return fail(LBM_EINVAL, "batch is NULL");
  if (id < 0 || id >= (int32_t)b->insts.size() || !b->insts[id].live)
    return fail(LBM_EINVAL, "no live instance with id %d", id);
  return LBM_OK;
}

int64_t completed_steps(const lbm_batch* b, const HostInst& h) {
  const int64_t t = std::min(b->clock, h.d.t_end);
  return std::max<int64_t>(0, t - h.d.t_start);
}

size_t used_extent(const lbm_batch* b) {
  size_t hi = 0;
  for (const HostInst& h : b->insts)
    if (h.live) hi = std::max(hi, (size_t)(h.d.off * (h.p.storage == LBM_STORE_F16 ? 2 : 4)) + h.bytes);
  return hi;
}

}  // namespace

extern "C" {

lbm_status lbm_batch_create(size_t arena_bytes, int32_t max_instances, int32_t max_tiles, int32_t graph_steps,
                            void* hip_stream, lbm_batch** out) {
  if (!out) return fail(LBM_EINVAL, "out is NULL");
  *out = nullptr;
  if (arena_bytes < 256 || max_instances < 1 || max_tiles < 1 || graph_steps < 1 || graph_steps > 4096)
    return fail(LBM_EINVAL, "bad batch sizes (arena %zu, instances %d, tiles %d, graph steps %d)", arena_bytes,
                max_instances, max_tiles, graph_steps);
  lbm_batch* b = new (std::nothrow) lbm_batch();
  if (!b) return fail(LBM_ENOMEM, "host allocation failed");
  grlbm::copy_users(1);
  auto bail = [&](lbm_status s) {
    lbm_batch_destroy(b);
    return s;
  };
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return bail(fail(LBM_EDEVICE, "no HIP device"));
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
    b->num_cus = cus;
  if (hip_stream) {
    b->stream = (hipStream_t)hip_stream;
  } else {
    if (hipStreamCreate(&b->stream) != hipSuccess) return bail(fail(LBM_EDEVICE, "hipStreamCreate failed"));
    b->own_stream = true;
  }
  b->arena_bytes = arena_bytes / 256 * 256;
  if (grlbm::dev_malloc((void**)&b->arena, b->arena_bytes) != hipSuccess)
    return bail(fail(LBM_ENOMEM, "hipMalloc of a %zu-byte arena failed", b->arena_bytes));
  b->free_list[0] = b->arena_bytes;
  b->max_inst = max_instances;
  b->max_tiles = max_tiles;
  if (grlbm::dev_malloc((void**)&b->d_insts, sizeof(BatchInst) * (size_t)max_instances) != hipSuccess ||
      grlbm::dev_malloc((void**)&b->d_tiles, sizeof(BatchTile) * (size_t)max_tiles * kGroups) != hipSuccess ||
      grlbm::dev_malloc((void**)&b->d_runs, sizeof(b->runs)) != hipSuccess ||
      grlbm::dev_malloc((void**)&b->d_scales, 5 * sizeof(unsigned)) != hipSuccess ||
      grlbm::dev_malloc((void**)&b->d_clock, sizeof(int64_t)) != hipSuccess ||
      grlbm::dev_malloc((void**)&b->d_flags, sizeof(int32_t) * (size_t)max_instances) != hipSuccess)
    return bail(fail(LBM_ENOMEM, "hipMalloc of the batch tables failed"));
  const int64_t zero = 0;
  if (hipMemcpyAsync(b->d_clock, &zero, sizeof zero, hipMemcpyHostToDevice, b->stream) != hipSuccess ||
      hipMemcpyAsync(b->d_runs, b->runs, sizeof(b->runs), hipMemcpyHostToDevice, b->stream) != hipSuccess ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return bail(fail(LBM_EDEVICE, "batch table initialisation failed"));
  b->graph_steps = graph_steps;
  // one 256-cell tile per block with plain loads and stores, at most 2 blocks per
  // CU: the fastest shape on a mixed FP32/FP16 serving load (persistent grids
  // trail it by 6-9%, the nontemporal hint by 5%; uncapped blocks by 1-2% in
  // solves/s, 4.5% on the 64 requests resident at once); lbm_batch_autotune picks
  // per workload
  b->tune.block = 256;
  b->tune.nontemporal = 0;
  b->tune.blocks_per_cu = 2;
  b->tune.grid = 0;
  b->spare.device = dev;
  b->spare.stream = b->stream;
  *out = b;
  return LBM_OK;
}

lbm_status lbm_batch_add(lbm_batch* b, const lbm_params* p, const double* Q, int64_t steps, int32_t* id) {
  if (!b || !p || !Q || !id) return fail(LBM_EINVAL, "NULL argument");
  if (steps < 0) return fail(LBM_EINVAL, "steps < 0");
  lbm_status st = grlbm::validate(p);
  if (st != LBM_OK) return st;
  st = grlbm::check_fields(p, Q);
  if (st != LBM_OK) return st;
  int32_t slot = -1;
  for (int32_t i = 0; i < (int32_t)b->insts.size(); ++i)
    if (!b->insts[i].live) {
      slot = i;
      break;
    }
  if (slot < 0) {
    if ((int32_t)b->insts.size() >= b->max_inst) return fail(LBM_ENOMEM, "batch holds %d instances already", b->max_inst);
    slot = (int32_t)b->insts.size();
    b->insts.emplace_back();
  }
  const int g = group_of(p);
  int64_t tiles_in_group = inst_tiles(p, b->tune.block);
  for (const HostInst& h : b->insts)
    if (h.live && h.group == g && h.d.t_end > b->clock) tiles_in_group += inst_tiles(&h.p, b->tune.block);
  if (tiles_in_group > b->max_tiles)
    return fail(LBM_ENOMEM, "instance needs %lld tiles beyond the capacity %d",
                (long long)inst_tiles(p, b->tune.block), b->max_tiles);
  const size_t bytes = grlbm::state_bytes(p);
  size_t off = 0;
  if (!arena_alloc(b, bytes, &off))
    return fail(LBM_ENOMEM, "arena has no free run of %zu bytes", bytes);
  HostInst& h = b->insts[slot];
  h.p = *p;
  h.bytes = bytes;
  h.group = g;
  h.d.c = grlbm::make_coll(p);
  h.d.g = grlbm::make_grid(p);
  const int el = p->storage == LBM_STORE_F16 ? 2 : 4;
  h.d.off = (int64_t)(off / el);
  h.d.t_start = b->clock;
  h.d.t_end = b->clock + steps;
  const int64_t N = (int64_t)p->nx * p->ny * p->nz;
  h.d.cells = (int32_t)grlbm::row_cells(h.d.g);
  h.d.inv_px = 1.0 / h.d.g.px;
  h.d.inv_ny = 1.0 / p->ny;
  // a second arena for what lies at the front of the first, where instances go first; the
  // first instance that can use it brings it, and its fields are staged there
  if (fast_way(h.p, h.d.g) != kSingle) prepare_fast(b, std::min(b->arena_bytes, kSpareFirst));
  const size_t field_bytes = sizeof(double) * 5 * (size_t)N;
  grlbm::Scratch dq(b->spare, field_bytes);
  if (!dq.p) {
    arena_free(b, off, bytes);
    return fail(LBM_ENOMEM, "staging allocation for the initial fields failed");
  }
  const double* Qd = (const double*)dq.p;
  hipError_t e = grlbm::copy_in(dq.p, Q, field_bytes, b->stream);
  if (e == hipSuccess && p->storage == LBM_STORE_F16) {
    st = grlbm::scales_from_fields(h.d.c, h.d.g, grlbm::make_init_coef(p), Qd, N, b->d_scales, b->stream);
    if (st != LBM_OK) {
      arena_free(b, off, bytes);
      return st;
    }
  }
  if (e == hipSuccess)
    e = grlbm::launch_init(b->arena + off, p->storage == LBM_STORE_F16, h.d.g, h.d.c, grlbm::make_init_coef(p), Qd,
                           N, b->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) {
    arena_free(b, off, bytes);
    return fail(LBM_EDEVICE, "instance initialisation failed: %s", hipGetErrorString(e));
  }
  h.live = true;
  h.pair_cus = 0;
  b->dirty = true;
  *id = slot;
  return LBM_OK;
}

lbm_status lbm_batch_run(lbm_batch* b, int64_t n) {
  if (!b) return fail(LBM_EINVAL, "batch is NULL");
  if (n < 0) return fail(LBM_EINVAL, "n < 0");
  try {
    return run_steps(b, n);
  } catch (const std::bad_alloc&) {  // the lists of a changed batch; nothing is enqueued yet
    return fail(LBM_ENOMEM, "host allocation of the tile lists failed");
  }
}

lbm_status lbm_batch_set_passes(lbm_batch* b, int32_t on) {
  if (!b) return fail(LBM_EINVAL, "batch is NULL");
  if (on != 0 && on != 1) return fail(LBM_EINVAL, "on = %d must be 0 or 1", on);
  lbm_status st = grlbm::switch_spare(b->spare, on != 0);
  if (st != LBM_OK) return st;
  drop_graphs(b);  // one names the second arena
  b->dirty = true;
  return LBM_OK;
}

lbm_status lbm_batch_get_passes(lbm_batch* b, int64_t* steps, int64_t* fast_steps, size_t* second_bytes) {
  if (!b) return fail(LBM_EINVAL, "batch is NULL");
  if (steps) *steps = b->clock;
  if (fast_steps) *fast_steps = b->fast_steps;
  const std::unique_lock<std::mutex> use = b->spare.hold();
  if (second_bytes) *second_bytes = b->spare.buf ? b->spare.bytes : 0;
  return LBM_OK;
}

lbm_status lbm_batch_query(lbm_batch* b, int32_t id, int64_t* done_steps, int32_t* finished) {
  lbm_status st = check_id(b, id);
  if (st != LBM_OK) return st;
  const HostInst& h = b->insts[id];
  if (done_steps) *done_steps = completed_steps(b, h);
  if (finished) *finished = h.d.t_end <= b->clock ? 1 : 0;
  return LBM_OK;
}

lbm_status lbm_batch_moments(lbm_batch* b, int32_t id, double* Q_out) {
  lbm_status st = check_id(b, id);
  if (st != LBM_OK) return st;
  if (!Q_out) return fail(LBM_EINVAL, "Q_out is NULL");
  st = check_kept(b);
  if (st != LBM_OK) return st;
  const HostInst& h = b->insts[id];
  const int64_t N = (int64_t)h.p.nx * h.p.ny * h.p.nz;
  const int el = h.p.storage == LBM_STORE_F16 ? 2 : 4;
  const size_t bytes = sizeof(double) * 5 * (size_t)N;
  grlbm::Scratch d(b->spare, bytes);
  if (!d.p) return fail(LBM_ENOMEM, "staging allocation for the moments failed");
  hipError_t e = grlbm::launch_gather(b->arena + (size_t)h.d.off * el, h.p.storage == LBM_STORE_F16, h.d.g, h.d.c, N,
                                      (completed_steps(b, h) & 1) != 0, 1, nullptr, (double*)d.p, b->stream);
  if (e == hipSuccess) e = grlbm::copy_out(Q_out, d.p, bytes, b->stream);
  if (e != hipSuccess) return fail(LBM_EDEVICE, "moments readout failed: %s", hipGetErrorString(e));
  return LBM_OK;
}

lbm_status lbm_batch_populations(lbm_batch* b, int32_t id, float* f_out, int64_t* step) {
  lbm_status st = check_id(b, id);
  if (st != LBM_OK) return st;
  if (!f_out) return fail(LBM_EINVAL, "f_out is NULL");
  st = check_kept(b);
  if (st != LBM_OK) return st;
  const HostInst& h = b->insts[id];
  const int64_t N = (int64_t)h.p.nx * h.p.ny * h.p.nz;
  const int el = h.p.storage == LBM_STORE_F16 ? 2 : 4;
  const size_t bytes = sizeof(float) * 35 * (size_t)N;
  grlbm::Scratch d(b->spare, bytes);
  if (!d.p) return fail(LBM_ENOMEM, "staging allocation for the populations failed");
  const int64_t done = completed_steps(b, h);
  hipError_t e = grlbm::launch_gather(b->arena + (size_t)h.d.off * el, h.p.storage == LBM_STORE_F16, h.d.g, h.d.c, N,
                                      (done & 1) != 0, 0, (float*)d.p, nullptr, b->stream);
  if (e == hipSuccess) e = grlbm::copy_out(f_out, d.p, bytes, b->stream);
  if (e != hipSuccess) return fail(LBM_EDEVICE, "population readout failed: %s", hipGetErrorString(e));
  if (step) *step = done;
  return LBM_OK;
}

lbm_status lbm_batch_nonfinite(lbm_batch* b, int32_t* ids, int32_t max, int32_t* count) {
  if (!b || !count) return fail(LBM_EINVAL, "NULL argument");
  if (max < 0 || (max > 0 && !ids)) return fail(LBM_EINVAL, "bad id buffer (max %d)", max);
  *count = 0;
  lbm_status st = check_kept(b);
  if (st != LBM_OK) return st;
  std::vector<grlbm::CheckItem> items;
  std::vector<int32_t> which;  // flag index -> instance id
  for (int32_t id = 0; id < (int32_t)b->insts.size(); ++id) {
    const HostInst& h = b->insts[id];
    if (!h.live) continue;
    const int32_t f16 = h.p.storage == LBM_STORE_F16 ? 1 : 0;
    for (int32_t c0 = 0; c0 < h.d.cells; c0 += grlbm::kCheckRun)
      items.push_back({h.d.off, h.d.g.S, c0, c0 + std::min(grlbm::kCheckRun, h.d.cells - c0), f16,
                       (int32_t)which.size(), h.d.g.nx, h.d.g.px});
    which.push_back(id);
  }
  const int32_t n = (int32_t)which.size();  // at most max_inst flags
  if (n == 0) return LBM_OK;
  if (items.size() > b->check_cap) {
    // no check kernel is in flight: every call ends synchronised
    const size_t want = std::max(items.size(), 2 * b->check_cap);
    if (b->d_check) (void)hipFree(b->d_check);
    b->d_check = nullptr;
    b->check_cap = 0;
    if (grlbm::dev_malloc((void**)&b->d_check, sizeof(grlbm::CheckItem) * want) != hipSuccess)
      return fail(LBM_ENOMEM, "hipMalloc of %zu check items failed", want);
    b->check_cap = want;
  }
  std::vector<int32_t> flags(n, 0);
  HIP_TRY(hipMemcpyAsync(b->d_check, items.data(), sizeof(grlbm::CheckItem) * items.size(), hipMemcpyHostToDevice,
                         b->stream));
  HIP_TRY(hipMemcpyAsync(b->d_flags, flags.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, b->stream));
  constexpr size_t kMaxGridY = 65535;
  for (size_t i0 = 0; i0 < items.size(); i0 += kMaxGridY) {
    const size_t m = std::min(kMaxGridY, items.size() - i0);
    hipLaunchKernelGGL(grlbm::k_batch_nonfinite, dim3(grlbm::kCheckBlocks, (unsigned)m), dim3(256), 0, b->stream,
                       (const char*)b->arena, b->d_check + i0, b->d_flags);
    HIP_TRY(hipGetLastError());
  }
  HIP_TRY(hipMemcpyAsync(flags.data(), b->d_flags, sizeof(int32_t) * n, hipMemcpyDeviceToHost, b->stream));
  // the host vectors above must outlive the copies
  HIP_TRY(hipStreamSynchronize(b->stream));
  for (int32_t i = 0; i < n; ++i) {
    if (!flags[i]) continue;
    if (*count < max) ids[*count] = which[i];
    ++*count;
  }
  return LBM_OK;
}

lbm_status lbm_batch_remove(lbm_batch* b, int32_t id) {
  lbm_status st = check_id(b, id);
  if (st != LBM_OK) return st;
  // work already enqueued may still touch the instance's memory
  HIP_TRY(hipStreamSynchronize(b->stream));
  HostInst& h = b->insts[id];
  const int el = h.p.storage == LBM_STORE_F16 ? 2 : 4;
  arena_free(b, (size_t)h.d.off * el, h.bytes);
  h.live = false;
  h.d.t_start = h.d.t_end = 0;  // stale tiles of a later run skip it
  b->dirty = true;
  return LBM_OK;
}

lbm_status lbm_batch_info(lbm_batch* b, lbm_batch_stats* out) {
  if (!b || !out) return fail(LBM_EINVAL, "NULL argument");
  std::memset(out, 0, sizeof *out);
  out->clock = b->clock;
  out->arena_bytes = b->arena_bytes;
  size_t freeb = 0, largest = 0;
  for (auto& kv : b->free_list) {
    freeb += kv.second;
    largest = std::max(largest, kv.second);
  }
  out->arena_free_bytes = freeb;
  out->arena_largest_free = largest;
  for (const HostInst& h : b->insts) {
    if (!h.live) continue;
    ++out->live_instances;
    if (h.d.t_end > b->clock) {
      ++out->active_instances;
      out->active_cells += (int64_t)h.p.nx * h.p.ny * h.p.nz;
    }
  }
  out->tuning = b->tune;
  out->graph_steps = b->graph_steps;
  return LBM_OK;
}

lbm_status lbm_batch_set_tuning(lbm_batch* b, const lbm_batch_tuning* t) {
  if (!b || !t) return fail(LBM_EINVAL, "NULL argument");
  if (t->block < 64 || t->block > 1024 || t->block % 64 != 0)
    return fail(LBM_EINVAL, "block = %d must be a multiple of 64 in [64, 1024]", t->block);
  if (t->grid < 0 || t->grid > (1 << 24)) return fail(LBM_EINVAL, "grid = %d outside [0, 2^24]", t->grid);
  if (t->blocks_per_cu < 0 || t->blocks_per_cu > 32) return fail(LBM_EINVAL, "blocks_per_cu outside [0, 32]");
  if (t->block != b->tune.block) {
    // the tile width is the block width: check the capacity before switching
    int64_t per_group[kGroups] = {0, 0, 0, 0};
    for (const HostInst& h : b->insts)
      if (h.live && h.d.t_end > b->clock) per_group[h.group] += inst_tiles(&h.p, t->block);
    for (int g = 0; g < kGroups; ++g)
      if (per_group[g] > b->max_tiles) return fail(LBM_ENOMEM, "block %d needs more tiles than the capacity", t->block);
  }
  b->tune = *t;
  b->tune.nontemporal = t->nontemporal ? 1 : 0;
  b->dirty = true;
  drop_graphs(b);
  return LBM_OK;
}

lbm_status lbm_batch_autotune(lbm_batch* b, int32_t trial_steps, lbm_batch_tuning* best, float* best_us,
                              lbm_batch_tuning* tried, float* tried_us, int32_t max_tried, int32_t* ntried) {
  if (!b || !best) return fail(LBM_EINVAL, "NULL argument");
  if (trial_steps < 2) return fail(LBM_EINVAL, "trial_steps must be >= 2");
  if (ntried) *ntried = 0;
  HIP_TRY(hipStreamSynchronize(b->stream));
  // snapshot of the live state: trials advance the instances, the snapshot puts
  // them back (results never depend on the launch shape)
  const size_t extent = used_extent(b);
  char* snap = nullptr;
  if (extent > 0) {
    if (grlbm::dev_malloc((void**)&snap, extent) != hipSuccess) return fail(LBM_ENOMEM, "snapshot of %zu bytes failed", extent);
    HIP_TRY(hipMemcpyAsync(snap, b->arena, extent, hipMemcpyDeviceToDevice, b->stream));
  }
  const lbm_batch_tuning orig = b->tune;
  const int64_t clock0 = b->clock;
  std::vector<lbm_batch_tuning> cands;
  for (int block : {128, 256, 512, 1024})
    for (int waves_per_cu : {8, 16, 32}) {
      const int bpc = std::max(1, waves_per_cu / (block / 64));
      if (bpc * (block / 64) != waves_per_cu) continue;
      for (int nt : {0, 1}) {
        lbm_batch_tuning t{};
        t.block = block;
        t.nontemporal = nt;
        t.blocks_per_cu = bpc;
        t.grid = b->num_cus * bpc;
        cands.push_back(t);
      }
    }
  // one block per tile, occupancy set by the registers alone, and for 256- and
  // 512-thread blocks capped at 8 or 16 waves per CU as well (the default shape
  // is one of these; nontemporal access with 4 blocks of 256 per CU runs large
  // cubes at the single-context rate)
  for (int block : {128, 256, 512, 1024})
    for (int bpc : {0, 2, 4})
      for (int nt : {0, 1}) {
        if (bpc > 0 && (block < 256 || block > 512 || bpc * (block / 64) > 16)) continue;
        lbm_batch_tuning t{};
        t.block = block;
        t.nontemporal = nt;
        t.blocks_per_cu = bpc;
        t.grid = 0;
        cands.push_back(t);
      }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  lbm_status st = LBM_OK;
  float best_time = 1e30f;
  lbm_batch_tuning best_t = orig;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    st = fail(LBM_EDEVICE, "event creation failed");
  }
  b->single_steps = true;
  for (size_t ci = 0; st == LBM_OK && ci < cands.size(); ++ci) {
    st = lbm_batch_set_tuning(b, &cands[ci]);
    if (st == LBM_ENOMEM) {  // this block width does not fit the tile capacity
      st = LBM_OK;
      continue;
    }
    if (st != LBM_OK) break;
    // warm-up: uploads the tiles for this width and captures the graph, so the timed
    // run replays it without host work in between
    st = run_steps(b, std::max(2, b->graph_steps));
    if (st != LBM_OK) break;
    float ms = 0.0f;
    if (hipEventRecord(e0, b->stream) != hipSuccess) { st = fail(LBM_EDEVICE, "event record failed"); break; }
    st = run_steps(b, trial_steps);
    if (st != LBM_OK) break;
    if (hipEventRecord(e1, b->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
      st = fail(LBM_EDEVICE, "trial timing failed");
      break;
    }
    const float us = ms * 1000.0f / trial_steps;
    if (tried && ntried && *ntried < max_tried) {
      tried[*ntried] = cands[ci];
      if (tried_us) tried_us[*ntried] = us;
      ++*ntried;
    }
    if (us < best_time) {
      best_time = us;
      best_t = cands[ci];
    }
    // restore the state and the clock
    if (extent > 0 && hipMemcpyAsync(b->arena, snap, extent, hipMemcpyDeviceToDevice, b->stream) != hipSuccess) {
      st = fail(LBM_EDEVICE, "snapshot restore failed");
      break;
    }
    b->clock = clock0;
    if (hipMemcpyAsync(b->d_clock, &b->clock, sizeof(int64_t), hipMemcpyHostToDevice, b->stream) != hipSuccess ||
        hipStreamSynchronize(b->stream) != hipSuccess) {
      st = fail(LBM_EDEVICE, "clock restore failed");
      break;
    }
    b->dirty = true;
  }
  b->single_steps = false;
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (snap) {
    (void)hipStreamSynchronize(b->stream);
    (void)hipFree(snap);
  }
  if (st != LBM_OK) return st;
  st = lbm_batch_set_tuning(b, &best_t);
  if (st != LBM_OK) return st;
  *best = best_t;
  if (best_us) *best_us = best_time;
  return LBM_OK;
}

lbm_status lbm_batch_destroy(lbm_batch* b) {
  if (!b) return LBM_OK;
  lbm_status st = LBM_OK;
  if (b->stream && hipStreamSynchronize(b->stream) != hipSuccess)
    st = fail(LBM_EDEVICE, "stream synchronisation failed during destroy");
  drop_graphs(b);
  grlbm::drop_spare(b->spare);
  if (b->arena) (void)hipFree(b->arena);
  if (b->d_insts) (void)hipFree(b->d_insts);
  if (b->d_tiles) (void)hipFree(b->d_tiles);
  if (b->d_multi) (void)hipFree(b->d_multi);
  if (b->d_runs) (void)hipFree(b->d_runs);
  if (b->d_clock) (void)hipFree(b->d_clock);
  if (b->d_check) (void)hipFree(b->d_check);
  if (b->d_flags) (void)hipFree(b->d_flags);
  if (b->d_scales) (void)hipFree(b->d_scales);
  if (b->own_stream && b->stream) (void)hipStreamDestroy(b->stream);
  delete b;
  grlbm::copy_users(-1);
  return st;
}

}  // extern "C"
