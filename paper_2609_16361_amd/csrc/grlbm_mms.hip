// grlbm_mms.hip -- GENERATED by paper_2609_16361_amd/mms_codegen.py; do not edit.
//
// Source S = dQ/dt + div Phi of eq. 1 for the manufactured solution of Sec. 3.1
// (eq. 8) under the flux of eq. 2 with constant mu and kappa, in lattice units, from
// a symbolic differentiation.  One lane per cell of an nx * ny * nz lattice (cell
// (i, j, l) at x = (i, j, l)), evaluated in FP64 and stored as FP32 in S[5][N].
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/grlbm_mms.h"
#include "grlbm_internal.h"

namespace {

// A block of 4 waves takes a tile of 64 x 8 x tz cells, a wave one row of 64 at a time.
// Every sine and cosine depends on one coordinate: one wave per axis evaluates the
// tile's, into LDS, and a cell needs about 350 FP64 operations besides (squares are
// products: pow(x, 2) is not simplified in FP64 and was half of the work).  Bound by
// FP64 issue and its latency.  On MI355X 128^3 took 229 us with all of it evaluated per
// cell, 130 us with pow, 36 us now; 64^3 35 and 9 us, 24^3 11 and 6 us.
constexpr int TX = 64, TY = 8, TZ = 4;  // tz is at most TZ

__device__ __forceinline__ double sq(double v) { return v * v; }

__global__ void __launch_bounds__(256, 3) k_mms_source(lbm_mms m, int32_t nx, int32_t ny, int32_t nz, int32_t tz,
                                                        double t, float* __restrict__ S) {
  __shared__ double vx[12][TX], vy[9][TY], vz[14][TZ];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
  const int r = (int)(blockIdx.x / ntx);
  const int x0 = (int)(blockIdx.x % ntx) * TX, y0 = (r % nty) * TY, z0 = (r / nty) * tz;
  const int i = lane;
  if (wave == 0) {
    const double x = (double)(x0 + i);
    const double e1 = m.W*t;
    const double e5 = m.K*x;
    const double e6 = cos(e5);
    const double e10 = e5 + 2.0/5.0;
    const double e11 = cos(e10);
    const double e20 = e1 + e5;
    const double e21 = sin(e20);
    const double e23 = sin(e10);
    const double e24 = sin(e5);
    const double e31 = e5 + 6.0/5.0;
    const double e32 = sin(e31);
    const double e33 = e32*m.P0;
    const double e55 = (21.0/20000.0)*e23;
    const double e62 = cos(e20);
    const double e67 = 7*e23;
    const double e73 = cos(e31);
    const double e86 = 400000*e33;
    vx[0][i] = e6;
    vx[1][i] = e11;
    vx[2][i] = e21;
    vx[3][i] = e23;
    vx[4][i] = e24;
    vx[5][i] = e32;
    vx[6][i] = e33;
    vx[7][i] = e55;
    vx[8][i] = e62;
    vx[9][i] = e67;
    vx[10][i] = e73;
    vx[11][i] = e86;
  } else if (wave == 1 && i < TY) {
    const double y = (double)(y0 + i);
    const double e1 = m.W*t;
    const double e35 = sq(m.U);
    const double e40 = e35*m.rho0;
    const double e41 = e40*m.K;
    const double e8 = m.K*y;
    const double e9 = sin(e8);
    const double e14 = e8 + 9.0/10.0;
    const double e15 = sin(e14);
    const double e25 = cos(e8);
    const double e30 = cos(e14);
    const double e42 = (9.0/20000.0)*e41*e9;
    const double e48 = e1 + e8;
    const double e49 = cos(e48);
    const double e68 = 7*e30;
    const double e74 = sin(e48);
    const double e84 = 240000*e49*m.P0;
    vy[0][i] = e9;
    vy[1][i] = e15;
    vy[2][i] = e25;
    vy[3][i] = e30;
    vy[4][i] = e42;
    vy[5][i] = e49;
    vy[6][i] = e68;
    vy[7][i] = e74;
    vy[8][i] = e84;
  } else if (wave == 2 && i < tz) {
    const double z = (double)(z0 + i);
    const double e1 = m.W*t;
    const double e35 = sq(m.U);
    const double e38 = m.U*m.W*m.rho0;
    const double e39 = (3.0/50.0)*e38;
    const double e40 = e35*m.rho0;
    const double e41 = e40*m.K;
    const double e43 = (3.0/10000.0)*e41;
    const double e76 = 80000*m.P0;
    const double e0 = m.K*z;
    const double e2 = e0 + e1;
    const double e3 = sin(e2);
    const double e4 = 4*e3;
    const double e13 = cos(e0);
    const double e18 = e0 + 17.0/10.0;
    const double e19 = cos(e18);
    const double e26 = cos(e2);
    const double e29 = sin(e18);
    const double e47 = (3.0/4000.0)*e29;
    const double e51 = e3*e39;
    const double e52 = e3*e43;
    const double e56 = sin(e0);
    const double e58 = e0 + 3.0/5.0;
    const double e59 = cos(e58);
    const double e69 = 5*e29;
    const double e72 = sin(e58);
    const double e87 = e59*e76;
    vz[0][i] = e3;
    vz[1][i] = e4;
    vz[2][i] = e13;
    vz[3][i] = e19;
    vz[4][i] = e26;
    vz[5][i] = e29;
    vz[6][i] = e47;
    vz[7][i] = e51;
    vz[8][i] = e52;
    vz[9][i] = e56;
    vz[10][i] = e59;
    vz[11][i] = e69;
    vz[12][i] = e72;
    vz[13][i] = e87;
  }
  __syncthreads();
  if (x0 + lane >= nx) return;
  const int64_t N = (int64_t)nx * ny * nz;
  const double e7 = 200*m.a;
  const double e17 = m.K*m.U;
  const double e34 = sq(m.K);
  const double e35 = sq(m.U);
  const double e38 = m.U*m.W*m.rho0;
  const double e39 = (3.0/50.0)*e38;
  const double e40 = e35*m.rho0;
  const double e41 = e40*m.K;
  const double e43 = (3.0/10000.0)*e41;
  const double e60 = e34*m.mu;
  const double e61 = e60*m.U;
  const double e65 = e35*e60;
  const double e66 = (1.0/(m.gamma - 1));
  const double e76 = 80000*m.P0;
  const double e6 = vx[0][lane];
  const double e11 = vx[1][lane];
  const double e21 = vx[2][lane];
  const double e23 = vx[3][lane];
  const double e24 = vx[4][lane];
  const double e32 = vx[5][lane];
  const double e33 = vx[6][lane];
  const double e55 = vx[7][lane];
  const double e62 = vx[8][lane];
  const double e67 = vx[9][lane];
  const double e73 = vx[10][lane];
  const double e86 = vx[11][lane];
  for (int row = wave; row < TY * tz; row += 4) {
    const int jy = row % TY, jz = row / TY;
    if (y0 + jy >= ny || z0 + jz >= nz) continue;
    const int64_t n = x0 + lane + (int64_t)nx * (y0 + jy + (int64_t)ny * (z0 + jz));
    const double e9 = vy[0][jy];
    const double e15 = vy[1][jy];
    const double e25 = vy[2][jy];
    const double e30 = vy[3][jy];
    const double e42 = vy[4][jy];
    const double e49 = vy[5][jy];
    const double e68 = vy[6][jy];
    const double e74 = vy[7][jy];
    const double e84 = vy[8][jy];
    const double e3 = vz[0][jz];
    const double e4 = vz[1][jz];
    const double e13 = vz[2][jz];
    const double e19 = vz[3][jz];
    const double e26 = vz[4][jz];
    const double e29 = vz[5][jz];
    const double e47 = vz[6][jz];
    const double e51 = vz[7][jz];
    const double e52 = vz[8][jz];
    const double e56 = vz[9][jz];
    const double e59 = vz[10][jz];
    const double e69 = vz[11][jz];
    const double e72 = vz[12][jz];
    const double e87 = vz[13][jz];
    const double e12 = 7*e11 + e7 + 5*e9;
    const double e16 = 5*e13 + 7*e15 + e7;
    const double e22 = 5*e19 + 3*e21 + e7;
    const double e27 = 5*e24 + 3*e25 + 2*e26 + 100;
    const double e28 = e17*e27;
    const double e36 = sq(e12);
    const double e37 = e12*e3;
    const double e44 = e27*e40;
    const double e45 = e44*m.K;
    const double e46 = e12*e45;
    const double e50 = sq(e16);
    const double e53 = e16*e22;
    const double e54 = e16*e45;
    const double e57 = e22*e45;
    const double e63 = sq(e22);
    const double e64 = e22*e29;
    const double e70 = e40*(e36 + e50 + e63);
    const double e71 = e3*e70;
    const double e75 = 2*e72 + 5*e73 + 3*e74 + 100;
    const double e77 = e75*e76;
    const double e78 = e27*e70 + e66*e77 + e77;
    const double e79 = e17*e78;
    const double e80 = (1.0/(e27));
    const double e81 = e75*e80;
    const double e82 = e75/sq(e27);
    const double e83 = e34*e80*m.P0*m.kappa/m.rho0;
    const double e85 = 2*e44;
    S[0 * N + n] = (float)((1.0/200.0)*m.rho0*((1.0/20.0)*e12*e6*m.K*m.U - 3.0/100.0*e16*e17*e9 - 1.0/50.0*e17*e22*e3 - 7.0/100.0*e23*e28 + (7.0/100.0)*e27*e30*m.K*m.U - 1.0/20.0*e28*e29 - e4*m.W));
    S[1 * N + n] = (float)((7.0/150.0)*e11*e34*m.U*m.mu - 1.0/600.0*e12*e16*e42 + (7.0/4000000.0)*e12*e27*e30*e35*m.K*m.rho0 + (1.0/800000.0)*e16*e25*e27*e35*m.K*m.rho0 - 1.0/600.0*e22*e37*e43 - 7.0/2000000.0*e23*e46 - 1.0/20.0*e33*m.K + (1.0/40.0)*e34*e9*m.U*m.mu + (1.0/800000.0)*e35*e36*e6*m.K*m.rho0 - 1.0/600.0*e37*e39 - 1.0/600.0*e46*e47);
    S[2 * N + n] = (float)((1.0/800000.0)*e12*e16*e35*e6*m.K*m.rho0 + (1.0/40.0)*e13*e34*m.U*m.mu + (7.0/150.0)*e15*e34*m.U*m.mu + (7.0/2000000.0)*e16*e27*e30*e35*m.K*m.rho0 - 1.0/600.0*e16*e51 - 1.0/600.0*e42*e50 - 1.0/600.0*e47*e54 + (3.0/100.0)*e49*m.K*m.P0 - 1.0/600.0*e52*e53 - 1.0/600.0*e54*e55 - 1.0/800000.0*e56*e57);
    S[3 * N + n] = (float)((1.0/800000.0)*e12*e22*e41*e6 + (1.0/30.0)*e19*e61 + (3.0/200.0)*e21*e61 - 1.0/600.0*e22*e51 + (3.0/20000.0)*e27*e38*e62 + (7.0/4000000.0)*e30*e57 - 1.0/600.0*e42*e53 - 1.0/400000.0*e45*e64 + (3.0/4000000.0)*e46*e62 - 1.0/600.0*e52*e63 - 1.0/600.0*e55*e57 + (1.0/50.0)*e59*m.K*m.P0);
    S[4 * N + n] = (float)((7.0/30000.0)*e11*e12*e34*e35*m.mu - 1.0/1600000000.0*e12*e17*(-5*e6*e70 + e66*e86 - e85*(-e12*e67 + 3*e22*e62) + e86) + (1.0/8000.0)*e12*e34*e35*e9*m.mu + (1.0/8000.0)*e13*e16*e34*e35*m.mu + (7.0/30000.0)*e15*e16*e34*e35*m.mu + (1.0/1600000000.0)*e16*m.K*m.U*(e66*e84 - 3*e70*e9 + e84 + e85*(5*e12*e25 + e16*e68)) + (1.0/6000.0)*e19*e22*e34*e35*m.mu + (3.0/40000.0)*e21*e22*e34*e35*m.mu + (3.0/4000000.0)*e22*e27*e35*e62*m.W*m.rho0 + (1.0/800000000.0)*e22*m.K*m.U*(-5*e44*(e16*e56 + e64) + e66*e87 - e71 + e87) - 7.0/60000.0*e23*e65*(14*e23 + e68 - e69) - 7.0/1600000000.0*e23*e79 - 1.0/1600.0*sq(e25)*e65 - 1.0/12000.0*e29*e65*(10*e29 - e67 + e68) - 1.0/320000000.0*e29*e79 - 7.0/60000.0*e30*e65*(14*e30 + e67 + e69) + (7.0/1600000000.0)*e30*e78*m.K*m.U + (3.0/100.0)*e49*e66*m.P0*m.W - 1.0/1600.0*sq(e56)*e65 - 9.0/40000.0*sq(e62)*e65 - 1.0/4000000.0*e71*m.W - 5*e83*(e24*e81 + 10*e32*e6*e80 + 10*sq(e6)*e82 - e73) - 3*e83*(e25*e81 + 6*e49*e80*e9 - e74 + 6*e82*sq(e9)) - 2*e83*(e26*e81 + 4*sq(e3)*e82 + e4*e59*e80 - e72));
  }
}

}  // namespace

extern "C" lbm_status lbm_mms_source(const lbm_mms* m, int32_t nx, int32_t ny, int32_t nz, double t,
                                     float* S_dev, void* hip_stream) {
  if (!m || !S_dev) return grlbm::fail(LBM_EINVAL, "constants or source array is NULL");
  if (nx < 1 || ny < 1 || nz < 1) return grlbm::fail(LBM_EINVAL, "empty lattice %d x %d x %d", nx, ny, nz);
  const int64_t N = (int64_t)nx * ny * nz;
  if (N > ((int64_t)1 << 31)) return grlbm::fail(LBM_EINVAL, "%lld cells exceed 2^31", (long long)N);
  // the thickest tiles that still give 512 blocks: thicker ones share more of the
  // sines and cosines (128^3: 36 us with 4 planes, 40 with 2), thinner ones leave a
  // wave fewer rows to do one after another (64^3: 8.9 us with 2 planes, 12.4 with 4)
  const int64_t xy = (((int64_t)nx + TX - 1) / TX) * (((int64_t)ny + TY - 1) / TY);
  int tz = TZ;
  while (tz > 1 && xy * (((int64_t)nz + tz - 1) / tz) < 512) tz /= 2;
  const int64_t tiles = xy * (((int64_t)nz + tz - 1) / tz);
  hipLaunchKernelGGL(k_mms_source, dim3((unsigned)tiles), dim3(256), 0, (hipStream_t)hip_stream, *m, nx, ny, nz, tz,
                     t, S_dev);
  HIP_TRY(hipGetLastError());
  return LBM_OK;
}
