// grlbm_pair.hip -- two time steps per pass over memory (k_step_pair) and the rule
// that picks its tiles.
//
// A single step moves every population in and out of HBM once (280 B per cell in
// FP32) and is bound by that; its arithmetic takes under half of the time.  A pair
// step reads the populations once, makes an odd and the following even AA step, and
// writes them once.  The odd parity holds f*_i(x), the populations after collision,
// at x itself (slot opposite(i)), so the pair is
//     gather f_i(x) = f*_i(x - c_i)         from buffer A (as the odd step reads)
//     f*   = collide(f)                     first collision
//     f'_i(x) = f*_i(x - c_i)               the step between, kept on the chip
//     f'*  = collide(f')                    second collision
//     store f'*                             to buffer B (as the even step stores)
// with the arithmetic of the single steps, so the results are theirs bit for bit.
// The second collision of a tile needs the first one on a layer of cells around it,
// which the tile computes as well from what it reads out of A; that is why a pair
// cannot run in place, and pairs alternate between the population buffer and a
// second one of the same size.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "grlbm_pair.hpp"

namespace grlbm {

template <int COLL, bool ZG, bool NTS>
__global__ void __launch_bounds__(kPairThreads) k_step_pair(const float* __restrict__ A, float* __restrict__ B,
                                                            Grid g, Coll c, PairTiles pt) {
  extern __shared__ float xs[];
  // blocks are dealt to the 8 XCDs in turn, and each XCD takes neighbouring tiles, whose
  // halos then meet in its L2
  const int xcd = (int)(blockIdx.x % 8), bi = (int)(blockIdx.x / 8);
  const int nxy = pt.ntx * pt.nty;
  int seg, xy;
  if (pt.by_plane) {  // all XCDs in the same z segment
    seg = bi / pt.per_xcd;
    xy = xcd * pt.per_xcd + (bi - seg * pt.per_xcd);
    if (xy >= nxy) return;
  } else {  // each XCD a run of tiles
    const int tile = xcd * pt.per_xcd + bi;
    if (tile >= nxy * pt.nseg) return;
    seg = tile / nxy;
    xy = tile - seg * nxy;
  }
  pair_update<COLL, ZG, NTS>(A, B, g, c, pt, seg, xy, xs);
}

// The tiles of a grid: the widths, heights and z segments that fit a block are priced
// and the cheapest is taken.  A round of a block (one plane of its tile) costs about
// the larger of two times, what its 128-byte lines take and what its waves' arithmetic
// and latency take.  Rows that do not start on a line touch one more, and a halo
// column touches a line per row.  A block makes lz + 2 rounds and pays about seven
// more to start and to drain; a CU holds one block, so a tile count just above a
// multiple of 256 costs a whole turn more (111^3 takes 252 tiles of 128 x 4 x 13).
// With several turns per CU, blocks that run on for long drift apart in z and lose
// what neighbours share (512^3, 128 x 4 tiles: 4005 us per step with 64-plane segments,
// 4376 with 128, 4599 with 512).  The weights were fitted to timings of 20 grids from
// 64^3 to 512^3 in up to 60 tilings each: the choice ran within 1% of the best on
// average, 3% at worst.  A tiling that leaves CUs free is preferred where it is nearly
// as fast: on small grids it makes fewer collisions twice, and other streams can use
// them (three contexts of 40^3 together: 3.0 us per step with 160 tiles of 40 x 10 x 1,
// 4.3 with 240 of 40 x 7 x 1, one alone 5.8 and 5.9).  With `share`, cus is a grid's part of a card that others fill.
PairTiles pair_tiles(const Grid& g, int cus, bool share) {
  PairTiles best{};
  double best_cost = 1e300;
  const int per = cus >= 8 ? cus / 8 : 1;  // blocks an XCD holds at once
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  auto price = [&](int w, int h) {
    const bool fullx = w >= g.nx, fully = h >= g.ny;
    const int halo = (fully ? 0 : 2 * w) + (fullx ? 0 : 2 * h);
    if (w * h > kPairCells || halo > kPairThreads - kPairCells) return;
    const bool lines = g.px % 32 == 0 && (w % 32 == 0 || fullx);
    const double row = w / 32.0 + (lines ? 0.0 : 1.0);
    const double reads = (h + (fully ? 0 : 2)) * row + (fullx ? 0.0 : 1.9 * h);
    const double memory = 8.7 * reads + 1.35 * h * row;
    const int64_t inner = up((int64_t)w * h, 64), outer = up(halo, 64);
    const double issue = inner + outer <= 4 ? 300.0 + 5.0 * (double)(inner + outer)  // a wave per SIMD
                                            : 333.0 + 1.5 * (double)(2 * inner + outer);
    const int ntx = (int)up(g.nx, w), nty = (int)up(g.ny, h);
    const int64_t nxy = (int64_t)ntx * nty;
    int nseg = 0;
    for (int lz = g.nz; lz >= 1; lz = (int)std::min<int64_t>(lz - 1, up(g.nz, nseg + 1))) {
      nseg = (int)up(g.nz, lz);
      if (nxy * nseg > 16ll * cus && nseg > 1) break;
      for (int by_plane : {0, 1}) {
        const int64_t per_xcd = by_plane ? up(nxy, 8) : up(nxy * nseg, 8);
        const int64_t turns = share ? up(nxy * nseg, cus) : up(by_plane ? per_xcd * nseg : per_xcd, per);
        const double filled = turns > 1 || share ? 1.0 : (double)(nxy * nseg) / (8.0 * per);
        const double m = memory * std::sqrt(filled);
        double cost = (double)turns * (lz + 9) * (std::max(m, issue) + 0.11 * std::min(m, issue));
        // the part of the card that other work could use meanwhile
        cost *= 1.0 + 0.25 * std::min(1.0, (double)(nxy * nseg) / (share ? cus : 8 * per));
        // tiles that cut aligned rows inside lines share the lines they store; beyond the
        // Infinity Cache those cross HBM in pieces (288^3: 1054 us with 72 x 7, 754 with 96 x 5)
        if (!lines && g.px % 32 == 0 && 140 * row_cells(g) >= (256ll << 20)) cost *= 1.25;
        if (turns > 1 && by_plane) cost *= 0.999;  // equal turns: all XCDs in one segment
        if (turns > 1 && lz > 64) cost *= 1.0 + 0.375 * std::min(2.0, lz / 128.0);
        if (cost < best_cost) {
          best_cost = cost;
          best.w = w;
          best.h = h;
          best.lz = lz;
          best.ntx = ntx;
          best.nty = nty;
          best.nseg = nseg;
          best.by_plane = by_plane;
          best.per_xcd = (int)per_xcd;
        }
      }
    }
  };
  int last = 0;
  for (int cap = g.nx < kPairCells ? g.nx : kPairCells; cap >= 1; --cap) {
    const int w = (int)up(g.nx, up(g.nx, cap));  // an even split into that many tiles
    if (w == last) continue;
    if (w < 24 && w < g.nx) break;
    last = w;
    for (int wa : {w, (w + 31) / 32 * 32}) {
      if (wa > kPairCells || (wa != w && wa >= g.nx)) continue;
      const int most = kPairCells / wa < g.ny ? kPairCells / wa : g.ny;
      int lasth = 0;
      for (int h = most; h >= 1 && 2 * h >= most; --h) {
        const int he = (int)up(g.ny, up(g.ny, h));
        if (he != lasth) price(wa, he);
        lasth = he;
      }
    }
  }
  return best;
}

// A pair of a single plane makes three first collisions per cell; it pays as long as
// launches dominate (1000 x 1000 x 1: 47.6 us per step in pairs, 43.2 in single steps;
// 100000 x 1 x 1: 5.5 against 8.6).  Every other grid measured ran faster in pairs, from
// 8^3 (3.4 against 4.0 us) to 512^3.
bool pair_worth(const Grid& g) { return g.nz > 1 || row_cells(g) < (1 << 18); }

hipError_t launch_pair(const StepLaunch& L, const PairTiles& p, const void* A, void* B, hipStream_t s) {
  const Grid& g = L.g;
  const dim3 grid((unsigned)(8 * p.per_xcd * (p.by_plane ? p.nseg : 1))), block(kPairThreads);
  const bool zg = g.zg_x || g.zg_y || g.zg_z;
  // nontemporal stores where they are whole lines of a state larger than the Infinity
  // Cache (256^3 449 against 482 us per step); else the hint costs: it drops what the
  // next pair would still find there (96^3 29.1 GLUP/s against 35.6 without), and a
  // line that two tiles share leaves the L2 in pieces (200^3 23.9 against 31.7)
  const bool nts = g.px % 32 == 0 && (p.w % 32 == 0 || p.w >= g.nx) && 140 * row_cells(g) >= (256ll << 20);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, kPairLds, s, (const float*)A, (float*)B, g, L.c, p);
    return hipGetLastError();
  };
  if (L.coll == 0) {
    if (zg) return nts ? go(k_step_pair<0, true, true>) : go(k_step_pair<0, true, false>);
    return nts ? go(k_step_pair<0, false, true>) : go(k_step_pair<0, false, false>);
  }
  if (zg) return nts ? go(k_step_pair<1, true, true>) : go(k_step_pair<1, true, false>);
  return nts ? go(k_step_pair<1, false, true>) : go(k_step_pair<1, false, false>);
}

}  // namespace grlbm
