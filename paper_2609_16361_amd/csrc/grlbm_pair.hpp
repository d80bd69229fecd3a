// grlbm_pair.hpp -- two time steps of one tile in one pass over memory (pair_update).
#pragma once
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

// An odd and the following even step of one tile, from A to B: column tile xy (of
// pt.ntx * pt.nty) and z segment seg.  Every lane of a block of kPairThreads calls this;
// xs holds kPairLds bytes.
//
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
// 256^3 the counters show 148 + 140 B).  One block of 13 waves per CU at 118-125
// registers; 5.3 TB/s, VALU 41% busy.  Measured on MI355X against two single steps
// (us per step): 256^3 794 -> 449, 128^3 99.8 -> 59, 111^3 59.8 -> 48.5, 96^3 37.8
// -> 25, 512^3 6845 -> 4100.  Loading the next plane ahead into registers gained
// nothing (472 against 462 us at 256^3: the loop-carried copies wait for the stores),
// 13 interior waves or two smaller blocks per CU ran 8-20% slower, and nontemporal
// loads lose the halo's reuse (736 us).
template <int COLL, bool ZG, bool NTS>
__device__ __forceinline__ void pair_update(const float* __restrict__ A, float* __restrict__ B, const Grid& g,
                                            const Coll& c, const PairTiles& pt, int seg, int xy, float* xs) {
  constexpr int NI = kPairCells + 64;  // interior cells and a column for the writes that leave the tile
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
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

}  // namespace grlbm
