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

#include "grlbm_device.hpp"
#include "grlbm_internal.h"

namespace grlbm {

// Element `byte` bytes past a base that is the same for the whole wave: one global
// access with a scalar base and a 32-bit offset per lane.
template <typename T>
__device__ __forceinline__ T* at_byte(T* base, uint32_t byte) {
  typedef __attribute__((address_space(1))) char gchar;
  gchar* b = (gchar*)wave_uniform(reinterpret_cast<uint64_t>(base));
  return (T*)(b + byte);
}
template <typename T>
__device__ __forceinline__ const T* at_byte(const T* base, uint32_t byte) {
  return at_byte(const_cast<T*>(base), byte);
}

// A block owns w x h columns of cells (w along x, h along y) and walks them along z
// from z0 to z1, one plane per round: the first collision on plane zz, then the
// second on plane zz - 1.  The 8 interior waves hold the tile's cells row by row and
// the halo waves the rows below and above and the columns left and right of it
// (no corners: D3Q7 has no diagonal velocities).  A lane keeps its column for the
// whole walk, so its addresses within a plane are computed once, and what moves
// along z (and the rest populations) stays in its registers: 15 floats.  The
// populations that move along x and y go through LDS, written at their destination
// cell, in two buffers by plane parity; so a round needs one barrier, which waits
// for LDS only and leaves loads and stores in flight.  The rounds before z0 and at
// z1 are the halo along z.  Along an axis the tile spans whole there is no halo and
// the writes wrap.
//
// Bound by HBM: 140 + 140 B per cell and pair, the halo's lines come from L2 (at
// 256^3 the counters show 145 + 140 B).  One block of 13 waves per CU at 118-125
// registers; 5.3 TB/s, VALU 41% busy.  Measured on MI355X against two single steps
// (us per step): 256^3 794 -> 449, 128^3 99.8 -> 59, 111^3 59.8 -> 48.5, 96^3 37.8
// -> 25, 512^3 6845 -> 4100.  Loading the next plane ahead into registers gained
// nothing (472 against 462 us at 256^3: the loop-carried copies wait for the stores),
// 13 interior waves or two smaller blocks per CU ran 8-20% slower, and nontemporal
// loads lose the halo's reuse (736 us).
template <int COLL, bool ZG, bool NTS>
__global__ void __launch_bounds__(kPairThreads) k_step_pair(const float* __restrict__ A, float* __restrict__ B,
                                                            Grid g, Coll c, PairTiles pt) {
  extern __shared__ float xs[];
  constexpr int NI = kPairCells + 64;  // interior cells and a column for the writes that leave the tile
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // the tile: blocks are dealt to the 8 XCDs in turn, and each XCD takes neighbouring
  // tiles, whose halos then meet in its L2
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
  const int ty = xy / pt.ntx, tx = xy - ty * pt.ntx;
  const int x0 = tx * pt.w, y0 = ty * pt.h;
  const int w = min(pt.w, g.nx - x0), h = min(pt.h, g.ny - y0);
  const int z0 = seg * pt.lz, z1 = min(g.nz, z0 + pt.lz);
  const bool fullx = w == g.nx, fully = h == g.ny;
  // this lane's cell (ex, ey) relative to the tile
  const bool iwave = wave < kPairCells / 64;
  const int nrow = fully ? 0 : 2 * w, nhalo = nrow + (fullx ? 0 : 2 * h);
  int ex, ey;
  bool act;
  if (iwave) {
    ey = t / w;
    ex = t - ey * w;
    act = ey < h;
  } else {
    int u = t - kPairCells;
    act = u < nhalo;
    if (u < nrow) {
      ey = u < w ? -1 : h;
      ex = u < w ? u : u - w;
    } else {
      u -= nrow;
      ex = u < h ? -1 : w;
      ey = u < h ? u : u - h;
    }
  }
  // beyond a zero-gradient face there is no cell; beyond a periodic one the other end
  int x = x0 + ex, y = y0 + ey;
  if (x < 0) {
    act = act && !(ZG && g.zg_x);
    x = g.nx - 1;
  } else if (x >= g.nx) {
    act = act && !(ZG && g.zg_x);
    x = 0;
  }
  if (y < 0) {
    act = act && !(ZG && g.zg_y);
    y = g.ny - 1;
  } else if (y >= g.ny) {
    act = act && !(ZG && g.zg_y);
    y = 0;
  }
  if (!act) {  // idle lanes load the tile's first column and store nothing
    x = x0;
    y = y0;
  }
  const bool inner = iwave && act;
  const bool wave_inner = iwave && 64 * wave < w * h;
  const bool wave_act = iwave ? wave_inner : 64 * wave - kPairCells < nhalo;
  const bool lo_x = ZG && g.zg_x && x == 0, hi_x = ZG && g.zg_x && x == g.nx - 1;
  const bool lo_y = ZG && g.zg_y && y == 0, hi_y = ZG && g.zg_y && y == g.ny - 1;
  // where the odd step reads f_i, as byte offsets within a plane; slots 1 and 2 are
  // taken from slot 1's array and 3 and 4 from slot 3's, the other slot lying S4 on
  const uint32_t S4 = 4u * (uint32_t)g.S;
  const int row = g.px * y;
  uint32_t oc = 4u * (uint32_t)(x + row);
  const uint32_t oxm = 4u * (uint32_t)((x == 0 ? g.nx - 1 : x - 1) + row);
  const uint32_t oxp = 4u * (uint32_t)((x == g.nx - 1 ? 0 : x + 1) + row);
  const uint32_t oym = 4u * (uint32_t)(x + g.px * (y == 0 ? g.ny - 1 : y - 1));
  const uint32_t oyp = 4u * (uint32_t)(x + g.px * (y == g.ny - 1 ? 0 : y + 1));
  uint32_t o1 = lo_x ? oc : S4 + oxm;
  uint32_t o2 = hi_x ? S4 + oc : oxp;
  uint32_t o3 = lo_y ? oc : S4 + oym;
  uint32_t o4 = hi_y ? S4 + oc : oyp;
  // LDS index of the tile's cell one step along (dx, dy), or the lane's own spare word
  const int spare = kPairCells + (t & 63);
  const int own = inner ? t : spare;
  auto target = [&](int dx, int dy) {
    int nx = ex + dx, ny = ey + dy;
    if (fullx && !(ZG && g.zg_x)) nx = nx < 0 ? w - 1 : (nx >= w ? 0 : nx);
    if (fully && !(ZG && g.zg_y)) ny = ny < 0 ? h - 1 : (ny >= h ? 0 : ny);
    return act && nx >= 0 && nx < w && ny >= 0 && ny < h ? ny * w + nx : spare;
  };
  const int wxp = target(1, 0), wxm = target(-1, 0), wyp = target(0, 1), wym = target(0, -1);
  const int64_t S = g.S, plane = (int64_t)g.px * g.ny;
  // the tile's first and last plane lie on a zero-gradient face: the ghost beyond
  // holds the plane's own populations
  const bool lo_ghost = ZG && g.zg_z && z0 == 0, hi_ghost = ZG && g.zg_z && z1 == g.nz;
  // f*: rest and f_{+z} of the last plane, f_{+z} of the one before; dn: f_{-z} of
  // the last plane (only a ghost needs it later)
  float rest[kFields], up1[kFields], up2[kFields], dn[ZG ? kFields : 1];
#pragma unroll 1
  for (int zz = z0 - 1; zz <= z1; ++zz) {
    float* wbuf = xs + (zz & 1) * (20 * NI);
    const float* rbuf = xs + ((zz + 1) & 1) * (20 * NI);
    if (wave_act && (iwave || (zz >= z0 && zz < z1))) {
      // keeps the offsets' widening beside the accesses, which lets them take the
      // scalar-base form
      asm volatile("" : "+v"(oc), "+v"(o1), "+v"(o2), "+v"(o3), "+v"(o4));
      float f[kPop];
      {
        const int z = zz < 0 ? g.nz - 1 : (zz >= g.nz ? 0 : zz);
        const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z == g.nz - 1 ? 0 : z + 1;
        const bool lo_z = ZG && g.zg_z && z == 0, hi_z = ZG && g.zg_z && z == g.nz - 1;
#pragma unroll
        for (int k = 0; k < kFields; ++k) {
          const float* Fk = A + (int64_t)(7 * k) * S;
          const float* Fz = Fk + plane * z;
          f[7 * k + 0] = ld<float, false>(at_byte(Fz, oc));
          f[7 * k + 1] = ld<float, false>(at_byte(Fz + S, o1));
          f[7 * k + 2] = ld<float, false>(at_byte(Fz + S, o2));
          f[7 * k + 3] = ld<float, false>(at_byte(Fz + 3 * S, o3));
          f[7 * k + 4] = ld<float, false>(at_byte(Fz + 3 * S, o4));
          f[7 * k + 5] = ld<float, false>(at_byte(lo_z ? Fk + 5 * S + plane * z : Fk + 6 * S + plane * zm, oc));
          f[7 * k + 6] = ld<float, false>(at_byte(hi_z ? Fk + 6 * S + plane * z : Fk + 5 * S + plane * zp, oc));
        }
      }
      collide<COLL, false>(f, c, nullptr);
#pragma unroll
      for (int k = 0; k < kFields; ++k) {
        wbuf[(0 * kFields + k) * NI + wxp] = f[7 * k + 1];
        wbuf[(1 * kFields + k) * NI + wxm] = f[7 * k + 2];
        wbuf[(2 * kFields + k) * NI + wyp] = f[7 * k + 3];
        wbuf[(3 * kFields + k) * NI + wym] = f[7 * k + 4];
        if constexpr (ZG) {
          // the ghost copies that enter through a zero-gradient face
          if (lo_x) wbuf[(0 * kFields + k) * NI + own] = f[7 * k + 1];
          if (hi_x) wbuf[(1 * kFields + k) * NI + own] = f[7 * k + 2];
          if (lo_y) wbuf[(2 * kFields + k) * NI + own] = f[7 * k + 3];
          if (hi_y) wbuf[(3 * kFields + k) * NI + own] = f[7 * k + 4];
        }
      }
      if (wave_inner) {
        float q[kPop];  // f' of plane zz - 1
#pragma unroll
        for (int k = 0; k < kFields; ++k) {
          q[7 * k] = rest[k];
          q[7 * k + 5] = up2[k];
          q[7 * k + 6] = f[7 * k + 6];
          if constexpr (ZG) {
            if (hi_ghost && zz == z1) q[7 * k + 6] = dn[k];
            dn[k] = f[7 * k + 6];
            if (lo_ghost && zz == z0) up1[k] = f[7 * k + 5];
          }
          up2[k] = up1[k];
          up1[k] = f[7 * k + 5];
          rest[k] = f[7 * k];
        }
        if (zz > z0) {
#pragma unroll
          for (int k = 0; k < kFields; ++k) {
            q[7 * k + 1] = rbuf[(0 * kFields + k) * NI + own];
            q[7 * k + 2] = rbuf[(1 * kFields + k) * NI + own];
            q[7 * k + 3] = rbuf[(2 * kFields + k) * NI + own];
            q[7 * k + 4] = rbuf[(3 * kFields + k) * NI + own];
          }
          collide<COLL, false>(q, c, nullptr);
          if (inner) {
            const int z = zz - 1;
            float* Bz = B + plane * z;
            const bool lo_z = ZG && g.zg_z && z == 0, hi_z = ZG && g.zg_z && z == g.nz - 1;
#pragma unroll
            for (int k = 0; k < kFields; ++k) {
              float* Fk = Bz + (int64_t)(7 * k) * S;
              const float* fo = q + 7 * k;
              st<float, NTS>(at_byte(Fk, oc), fo[0]);
              st<float, NTS>(at_byte(Fk + 1 * S, oc), lo_x ? fo[1] : fo[2]);
              st<float, NTS>(at_byte(Fk + 2 * S, oc), hi_x ? fo[2] : fo[1]);
              st<float, NTS>(at_byte(Fk + 3 * S, oc), lo_y ? fo[3] : fo[4]);
              st<float, NTS>(at_byte(Fk + 4 * S, oc), hi_y ? fo[4] : fo[3]);
              st<float, NTS>(at_byte(Fk + 5 * S, oc), lo_z ? fo[5] : fo[6]);
              st<float, NTS>(at_byte(Fk + 6 * S, oc), hi_z ? fo[6] : fo[5]);
            }
          }
        }
      }
    }
    __syncthreads();
  }
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
// average, 3% at worst.
PairTiles pair_tiles(const Grid& g, int cus) {
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
    const double issue = 333.0 + 1.5 * (double)(2 * up((int64_t)w * h, 64) + up(halo, 64));
    const int ntx = (int)up(g.nx, w), nty = (int)up(g.ny, h);
    const int64_t nxy = (int64_t)ntx * nty;
    int nseg = 0;
    for (int lz = g.nz; lz >= 1; lz = (int)std::min<int64_t>(lz - 1, up(g.nz, nseg + 1))) {
      nseg = (int)up(g.nz, lz);
      if (nxy * nseg > 16ll * cus && nseg > 1) break;
      for (int by_plane : {0, 1}) {
        const int64_t per_xcd = by_plane ? up(nxy, 8) : up(nxy * nseg, 8);
        const int64_t turns = up(by_plane ? per_xcd * nseg : per_xcd, per);
        const double filled = turns > 1 ? 1.0 : (double)(nxy * nseg) / (8.0 * per);
        const double m = memory * std::sqrt(filled);
        double cost = (double)turns * (lz + 9) * (std::max(m, issue) + 0.11 * std::min(m, issue));
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
  const int lds = 2 * 20 * (kPairCells + 64) * (int)sizeof(float);
  const bool zg = g.zg_x || g.zg_y || g.zg_z;
  // nontemporal stores where they are whole lines of a state larger than the Infinity
  // Cache (256^3 449 against 482 us per step); else the hint costs: it drops what the
  // next pair would still find there (96^3 29.1 GLUP/s against 35.6 without), and a
  // line that two tiles share leaves the L2 in pieces (200^3 23.9 against 31.7)
  const bool nts = g.px % 32 == 0 && (p.w % 32 == 0 || p.w >= g.nx) && 140 * row_cells(g) >= (256ll << 20);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, lds, s, (const float*)A, (float*)B, g, L.c, p);
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
