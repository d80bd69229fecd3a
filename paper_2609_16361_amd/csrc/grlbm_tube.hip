// grlbm_tube.hip -- k_step_tube, up to ten time steps of a tube per launch, and the rule
// that picks its window and step count.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "grlbm_tube.hpp"

namespace grlbm {

// One block per window of a tube (tube_update).  On a long tube bound by VALU issue (the
// window's ends are computed and dropped) and HBM together, on a short one by the
// latency of a step in one wave per SIMD and of the launch.  Measured on MI355X, us per
// step of a context on its own stream, 4 x 4 cross-section, single steps before -> now:
// FP32 256 columns 4.3 -> 1.8, 4097 7.7 -> 3.0, 283000 (4.5 M cells) 230 -> 98; FP16 256
// columns 4.4 -> 2.7, 4097 5.8 -> 4.1, 283000 117 -> 106.
template <int COLL, typename T, int L>
__global__ void __launch_bounds__(L, 4) k_step_tube(const T* __restrict__ A, T* __restrict__ B, Grid g, Coll c,
                                                     TubeShape sh, int steps, int64_t t0) {
  extern __shared__ float xs[];
  tube_update<COLL, T, L>(A, B, g, c, (int)blockIdx.x * sh.inner, sh.width, sh.inner, steps, t0, xs);
}

// Blocks have 256 or 512 lanes (4 or 2 on a CU at 92-111 registers and 30 or 60 KB of
// LDS).  A step takes 0.55 + 0.56 w us with w waves per SIMD (FP16, whose stores round:
// 1.45 + 0.65 w), a launch 3.6 us besides, and on a full card a turn of blocks moves its
// windows through HBM at 8 TB/s, counted in whole lines, partly under the other blocks'
// arithmetic.  Within 20% of the timings over tubes of 256 to 283000 columns with
// cross-sections of 1 to 25 cells.
double tube_lines(int64_t cross, int width, bool f16) { return (double)cross * ((width - 1) * (f16 ? 2.0 : 4.0) + 128.0); }

double tube_price(const TubeShape& sh, double lines, int64_t blocks, bool f16, int cus) {
  const int resident = 1024 / sh.lanes;
  const int64_t slots = (int64_t)cus * resident;
  const double turns = (double)((blocks + slots - 1) / slots);
  const double waves = (double)std::min<int64_t>(resident, (blocks + cus - 1) / cus) * sh.lanes / 256.0;
  const double issue = sh.steps * (f16 ? 1.45 + 0.65 * waves : 0.55 + 0.56 * waves);
  const double memory = 70.0 * lines * (double)std::min<int64_t>(blocks, slots) / 8.0e6;
  return (3.6 + turns * (std::max(issue, memory) + 0.25 * std::min(issue, memory))) / sh.steps;
}

// The window and the most steps per launch of a tube, by the estimated time per step
// (lanes = 0: none, the grid is no tube or steps faster otherwise).  More steps per
// launch share the launch but drop more columns.  Against them stand the other ways to
// step: pairs (FP32, about 4.5 us + cells / 28500 us) and single steps (FP16, 4.4 us +
// cells / 58000 us, or cells / 37500 us beyond the caches; a tenth is left for the
// estimate's error).  Windows of cross-sections over 25 cells lose too much to their
// ends (FP32 8 x 4 cells, 4097 columns: 11.4 us per step, 8.7 in pairs).
TubeShape tube_shape(const Grid& g, bool f16, int cus) {
  TubeShape best{};
  const int64_t cross = (int64_t)g.ny * g.nz;
  if (cross > kTubeCross) return best;
  const double cells = (double)cross * g.nx;
  double best_cost = f16 ? 0.9 * std::max(4.4 + cells / 58000.0, cells / 37500.0) : 4.5 + cells / 28500.0;
  for (int lanes : {256, 512}) {
    const int width = (int)(lanes / cross);
    for (int steps = 2; steps <= kTubeSteps && width - 2 * steps >= 2; steps += 2) {
      const TubeShape sh{lanes, width, width - 2 * steps, steps, 0};
      const double cost = tube_price(sh, tube_lines(cross, width, f16), (g.nx + sh.inner - 1) / sh.inner, f16, cus);
      if (cost < best_cost) {
        best_cost = cost;
        best = sh;
      }
    }
  }
  // A run shorter than its shape's launches loads windows for few steps.  Measured against
  // single steps at 4, 6, 8 and 10 steps: FP16 in 256-lane blocks 0.9 of their time at 4; in
  // 512-lane blocks 1.2-1.4, 1.0-1.1 (0.97 with up to six steps a launch) and 0.85-0.96 with
  // a block per CU, 1.5, 1.2, 1.05 and 0.96 with two; FP32 0.55-0.9 at 4 but 1.03-1.27 in
  // narrow windows (25 cells across) or several turns of blocks, and 0.75 at 6.
  const int64_t blocks = best.lanes ? (g.nx + best.inner - 1) / best.inner : 0;
  if (f16) {
    best.least = best.lanes == 256 ? 4 : (blocks > cus ? 10 : (best.steps > 6 ? 8 : 6));
  } else {
    best.least = cross > 20 || blocks > 2 * cus ? 6 : 4;
  }
  return best;
}

// Dynamic LDS of a block.  Up to two blocks per CU, the reservation keeps the hardware
// from putting more on a CU than even dealing gives.
int tube_lds(const TubeShape& sh, int64_t blocks, int cus) {
  const int need = 30 * (int)sizeof(float) * sh.lanes;
  const int apart = blocks <= cus ? 82 * 1024 : (blocks <= 2 * cus ? 55 * 1024 : 0);
  return std::max(need, apart);
}

hipError_t launch_tube(const StepLaunch& L, const TubeShape& sh, int cus, const void* A, void* B, int steps,
                       int64_t t0, hipStream_t s) {
  const int64_t blocks = (L.g.nx + sh.inner - 1) / sh.inner;
  auto go = [&](auto kernel, auto* a, auto* b) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(sh.lanes), tube_lds(sh, blocks, cus), s, a, b, L.g, L.c,
                       sh, steps, t0);
    return hipGetLastError();
  };
  auto typed = [&](auto* a, auto* b) {
    using T = std::remove_pointer_t<decltype(b)>;
    if (sh.lanes == 256)
      return L.coll == 0 ? go(k_step_tube<0, T, 256>, a, b) : go(k_step_tube<1, T, 256>, a, b);
    return L.coll == 0 ? go(k_step_tube<0, T, 512>, a, b) : go(k_step_tube<1, T, 512>, a, b);
  };
  if (L.f16) return typed((const _Float16*)A, (_Float16*)B);
  return typed((const float*)A, (float*)B);
}

}  // namespace grlbm
