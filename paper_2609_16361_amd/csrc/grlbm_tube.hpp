// grlbm_tube.hpp -- several time steps per pass over memory for tubes: grids whose
// cross-section (ny * nz cells) fits a block (tube_update).
#pragma once
#include "grlbm_device.hpp"
#include "grlbm_internal.h"

namespace grlbm {

// A population as the storage holds it.  FP16: rounded with the dither of the slot it
// is stored in, hc being the key of the cell (the value st_pop stores).
template <typename T>
__device__ __forceinline__ float as_stored(float v, uint32_t hc, int slot) {
  if constexpr (sizeof(T) == 2) {
    return static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)half_bits(v, hc, slot)));
  } else {
    return v;
  }
}

// K steps (K even, from an even step t0 of the instance on) of the window of W columns
// of one tube that starts K columns before x0, one cell per lane: lane t holds column
// t % W of cross-section cell t / W.  The state is at even parity, where slot i of a
// cell holds f_i, so loads and stores are the lane's own cell's; the populations stay
// in registers and the 30 moving ones are exchanged through LDS (xs, 30 * L floats).
// A step makes one more column at each end of the window depend on cells outside it;
// the I <= W - 2 K columns from x0 on remain right and are stored.  Values and, in FP16,
// their rounding after every step are those of the single steps: an even step rounds
// f*_i with the key of its own cell and the slot opposite to i, an odd step with the
// key of the downstream cell and slot i; ghost copies at zero-gradient faces are
// rounded with the cell's own key and slot i.
// L = blockDim.x; every lane calls this (barriers).
template <int COLL, typename T, int L>
__device__ __forceinline__ void tube_update(const T* __restrict__ A, T* __restrict__ B, const Grid& g,
                                            const Coll& c, int x0, int W, int I, int K, int64_t t0,
                                            float* xs) {
  const int t = threadIdx.x;
  const int cross = t / W, ex = t - cross * W;
  const int z = cross / g.ny, y = cross - z * g.ny;
  int x = x0 - K + ex;
  bool act = cross < g.ny * g.nz;
  if (g.zg_x) {
    act = act && x >= 0 && x < g.nx;
  } else {
    x %= g.nx;
    if (x < 0) x += g.nx;
  }
  const bool inner = act && ex >= K && ex < K + I && x0 - K + ex < g.nx;
  const bool lo_x = g.zg_x && x == 0, hi_x = g.zg_x && x == g.nx - 1;
  const bool lo_y = g.zg_y && y == 0, hi_y = g.zg_y && y == g.ny - 1;
  const bool lo_z = g.zg_z && z == 0, hi_z = g.zg_z && z == g.nz - 1;
  // the lane f_i comes from: the upstream cell's, or this one at a zero-gradient face
  // (and at the window's ends, whose values no stored cell depends on)
  const int cz = g.ny * W;
  const int s1 = (lo_x || ex == 0) ? t : t - 1;
  const int s2 = (hi_x || ex == W - 1) ? t : t + 1;
  const int s3 = lo_y ? t : (y == 0 ? t + (g.ny - 1) * W : t - W);
  const int s4 = hi_y ? t : (y == g.ny - 1 ? t - (g.ny - 1) * W : t + W);
  const int s5 = lo_z ? t : (z == 0 ? t + (g.nz - 1) * cz : t - cz);
  const int s6 = hi_z ? t : (z == g.nz - 1 ? t - (g.nz - 1) * cz : t + cz);
  const bool ghost[kQ] = {false, lo_x, hi_x, lo_y, hi_y, lo_z, hi_z};
  const int n = act ? x + g.px * cross : 0;
  float f[kPop];
  if (act) {
#pragma unroll
    for (int s = 0; s < kPop; ++s) f[s] = ld<T, false>(at(A + (int64_t)s * g.S, n));
  }
#pragma unroll 1
  for (int k = 0; k < K; ++k) {
    const bool odd = (k & 1) != 0;
    uint32_t hc = 0;
    if constexpr (sizeof(T) == 2) hc = cell_key(n, step_key(t0 + k));
    if (act) {
      collide<COLL, false, sizeof(T) == 2>(f, c, nullptr);
#pragma unroll
      for (int q = 0; q < kFields; ++q) {
        float* fo = f + 7 * q;
        float* w = xs + 6 * q * L + t;
        fo[0] = as_stored<T>(fo[0], hc, 7 * q);
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          const float v = fo[i];
          if (sizeof(T) == 2 && !odd) {
            w[(i - 1) * L] = as_stored<T>(v, hc, 7 * q + ((i - 1) ^ 1) + 1);
          } else {
            w[(i - 1) * L] = v;
          }
        }
      }
      if (sizeof(T) == 2 && !odd) {
        // ghost copies stay here, in their own slot's rounding
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          if (ghost[i]) {
#pragma unroll
            for (int q = 0; q < kFields; ++q) f[7 * q + i] = as_stored<T>(f[7 * q + i], hc, 7 * q + i);
          }
        }
      }
    }
    __syncthreads();
    if (act) {
#pragma unroll
      for (int q = 0; q < kFields; ++q) {
        float* fo = f + 7 * q;
        const float* r = xs + 6 * q * L;
        const float v[kQ] = {0.0f, r[s1], r[L + s2], r[2 * L + s3], r[3 * L + s4], r[4 * L + s5], r[5 * L + s6]};
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          if constexpr (sizeof(T) == 2) {
            fo[i] = !odd && ghost[i] ? fo[i] : v[i];
          } else {
            fo[i] = v[i];
          }
        }
      }
      if (sizeof(T) == 2 && odd) {
#pragma unroll
        for (int q = 0; q < kFields; ++q)
#pragma unroll
          for (int i = 1; i < kQ; ++i) f[7 * q + i] = as_stored<T>(f[7 * q + i], hc, 7 * q + i);
      }
    }
    __syncthreads();
  }
  if (inner) {
#pragma unroll
    for (int s = 0; s < kPop; ++s) st<T, false>(at(B + (int64_t)s * g.S, n), f[s]);
  }
}

}  // namespace grlbm
