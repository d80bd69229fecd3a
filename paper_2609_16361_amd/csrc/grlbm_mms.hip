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

// A block of 4 waves takes a tile of 64 x ty x tz cells, a wave one row of 64 at a time,
// all of its rows in one plane.  Every sine and cosine depends on one coordinate: one
// wave per axis evaluates the tile's, into LDS, with all else that depends on that
// coordinate alone (grouped by the generator); a lane keeps the values of its x and z
// and needs about 200 FP64 operations per cell besides (squares are products: pow(x, 2)
// is not simplified in FP64).  Bound by FP64 issue and its latency, at 188 registers.  On
// MI355X 128^3 took 229 us with all of it evaluated per cell, 34 us with the sines and
// cosines alone from LDS and about 350 operations per cell, 23 us now; 256^3 215 and 137
// us in the last two forms, 24^3 11 us, 5.4 and 5.1.  At 168 registers it spills (33 us);
// z values read per row instead of kept take 29 us.
constexpr int TX = 64, TY = 16, TZ = 4;  // ty is 8 or TY; tz is 1, 2 or TZ

__device__ __forceinline__ double sq(double v) { return v * v; }

__global__ void __launch_bounds__(256, 2) k_mms_source(lbm_mms m, int32_t nx, int32_t ny, int32_t nz, int32_t ty,
                                                        int32_t tz, double t, float* __restrict__ S) {
  __shared__ double vx[30][TX], vy[27][TY], vz[29][TZ];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntx = (nx + TX - 1) / TX, nty = (ny + ty - 1) / ty;
  const int r = (int)(blockIdx.x / ntx);
  const int x0 = (int)(blockIdx.x % ntx) * TX, y0 = (r % nty) * ty, z0 = (r / nty) * tz;
  const int i = lane;
  if (wave == 0) {
    const double x = (double)(x0 + i);
    const double e1 = m.W*t;
    const double e7 = 200*m.a;
    const double e34 = sq(m.K);
    const double e35 = sq(m.U);
    const double e38 = m.U*m.W*m.rho0;
    const double e40 = e35*m.rho0;
    const double e41 = e40*m.K;
    const double e60 = e34*m.mu;
    const double e61 = e60*m.U;
    const double e65 = e35*e60;
    const double e66 = (1.0/(m.gamma - 1));
    const double e5 = m.K*x;
    double e24, e6;
    sincos(e5, &e24, &e6);
    const double e10 = e5 + 2.0/5.0;
    double e23, e11;
    sincos(e10, &e23, &e11);
    const double g0 = 7*e11 + e7;
    const double e20 = e1 + e5;
    double e21, e62;
    sincos(e20, &e21, &e62);
    const double g4 = 3*e21 + e7;
    const double g6 = 5*e24 + 100;
    const double e31 = e5 + 6.0/5.0;
    double e32, e73;
    sincos(e31, &e32, &e73);
    const double e33 = e32*m.P0;
    const double e55 = (21.0/20000.0)*e23;
    const double e67 = 7*e23;
    const double g9 = 5*e73 + 100;
    const double e86 = 400000*e33;
    const double g13 = -7.0/100.0*e23;
    const double g17 = (1.0/20.0)*e6*m.K*m.U;
    const double g21 = -7.0/2000000.0*e23;
    const double g26 = (1.0/800000.0)*e35*e6*m.K*m.rho0;
    const double g29 = (7.0/150.0)*e11*e34*m.U*m.mu - 1.0/20.0*e33*m.K;
    const double g33 = -1.0/600.0*e55;
    const double g38 = (3.0/4000000.0)*e62;
    const double g40 = (3.0/20000.0)*e38*e62;
    const double g41 = (1.0/800000.0)*e41*e6;
    const double g42 = (3.0/200.0)*e21*e61;
    const double g44 = 10*sq(e6);
    const double g45 = 10*e32*e6;
    const double g46 = -e73;
    const double g53 = -7.0/1600000000.0*e23;
    const double g56 = 14*e23;
    const double g58 = -7.0/60000.0*e23*e65;
    const double g61 = -e67;
    const double g64 = 3*e62;
    const double g65 = -5*e6;
    const double g66 = e66*e86 + e86;
    const double g78 = (3.0/40000.0)*e21*e34*e35*m.mu;
    const double g79 = (7.0/30000.0)*e11*e34*e35*m.mu;
    const double g81 = (3.0/4000000.0)*e35*e62*m.W*m.rho0;
    const double g82 = -9.0/40000.0*sq(e62)*e65;
    vx[0][i] = g0;
    vx[1][i] = g4;
    vx[2][i] = e24;
    vx[3][i] = g6;
    vx[4][i] = e67;
    vx[5][i] = g9;
    vx[6][i] = g13;
    vx[7][i] = g17;
    vx[8][i] = g21;
    vx[9][i] = g26;
    vx[10][i] = g29;
    vx[11][i] = g33;
    vx[12][i] = g38;
    vx[13][i] = g40;
    vx[14][i] = g41;
    vx[15][i] = g42;
    vx[16][i] = g44;
    vx[17][i] = g45;
    vx[18][i] = g46;
    vx[19][i] = g53;
    vx[20][i] = g56;
    vx[21][i] = g58;
    vx[22][i] = g61;
    vx[23][i] = g64;
    vx[24][i] = g65;
    vx[25][i] = g66;
    vx[26][i] = g78;
    vx[27][i] = g79;
    vx[28][i] = g81;
    vx[29][i] = g82;
  } else if (wave == 1 && i < ty) {
    const double y = (double)(y0 + i);
    const double e1 = m.W*t;
    const double e7 = 200*m.a;
    const double e17 = m.K*m.U;
    const double e34 = sq(m.K);
    const double e35 = sq(m.U);
    const double e40 = e35*m.rho0;
    const double e41 = e40*m.K;
    const double e60 = e34*m.mu;
    const double e65 = e35*e60;
    const double e66 = (1.0/(m.gamma - 1));
    const double e8 = m.K*y;
    double e9, e25;
    sincos(e8, &e9, &e25);
    const double g1 = 5*e9;
    const double e14 = e8 + 9.0/10.0;
    double e15, e30;
    sincos(e14, &e15, &e30);
    const double g2 = 7*e15 + e7;
    const double g7 = 3*e25;
    const double e42 = (9.0/20000.0)*e41*e9;
    const double e48 = e1 + e8;
    double e74, e49;
    sincos(e48, &e74, &e49);
    const double e68 = 7*e30;
    const double g10 = 3*e74;
    const double e84 = 240000*e49*m.P0;
    const double g15 = -3.0/100.0*e17*e9;
    const double g18 = (7.0/100.0)*e30*m.K*m.U;
    const double g24 = -1.0/600.0*e42;
    const double g27 = (1.0/800000.0)*e25*e35*m.K*m.rho0;
    const double g28 = (7.0/4000000.0)*e30*e35*m.K*m.rho0;
    const double g30 = (1.0/40.0)*e34*e9*m.U*m.mu;
    const double g35 = (7.0/2000000.0)*e30*e35*m.K*m.rho0;
    const double g36 = (7.0/150.0)*e15*e34*m.U*m.mu + (3.0/100.0)*e49*m.K*m.P0;
    const double g39 = (7.0/4000000.0)*e30;
    const double g47 = 6*sq(e9);
    const double g48 = 6*e49*e9;
    const double g49 = -e74;
    const double g59 = 14*e30;
    const double g60 = -7.0/60000.0*e30*e65;
    const double g70 = 5*e25;
    const double g71 = -3*e9;
    const double g72 = e66*e84 + e84;
    const double g74 = (7.0/1600000000.0)*e30*m.K*m.U;
    const double g76 = (1.0/8000.0)*e34*e35*e9*m.mu;
    const double g80 = (7.0/30000.0)*e15*e34*e35*m.mu;
    const double g83 = -1.0/1600.0*sq(e25)*e65 + (3.0/100.0)*e49*e66*m.P0*m.W;
    vy[0][i] = g1;
    vy[1][i] = g2;
    vy[2][i] = e25;
    vy[3][i] = g7;
    vy[4][i] = e68;
    vy[5][i] = g10;
    vy[6][i] = g15;
    vy[7][i] = g18;
    vy[8][i] = g24;
    vy[9][i] = g27;
    vy[10][i] = g28;
    vy[11][i] = g30;
    vy[12][i] = g35;
    vy[13][i] = g36;
    vy[14][i] = g39;
    vy[15][i] = g47;
    vy[16][i] = g48;
    vy[17][i] = g49;
    vy[18][i] = g59;
    vy[19][i] = g60;
    vy[20][i] = g70;
    vy[21][i] = g71;
    vy[22][i] = g72;
    vy[23][i] = g74;
    vy[24][i] = g76;
    vy[25][i] = g80;
    vy[26][i] = g83;
  } else if (wave == 2 && i < tz) {
    const double z = (double)(z0 + i);
    const double e1 = m.W*t;
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
    const double e0 = m.K*z;
    const double e2 = e0 + e1;
    double e3, e26;
    sincos(e2, &e3, &e26);
    const double e4 = 4*e3;
    double e56, e13;
    sincos(e0, &e56, &e13);
    const double g3 = 5*e13;
    const double e18 = e0 + 17.0/10.0;
    double e29, e19;
    sincos(e18, &e29, &e19);
    const double g5 = 5*e19;
    const double g8 = 2*e26;
    const double e47 = (3.0/4000.0)*e29;
    const double e51 = e3*e39;
    const double e52 = e3*e43;
    const double e58 = e0 + 3.0/5.0;
    double e72, e59;
    sincos(e58, &e72, &e59);
    const double e69 = 5*e29;
    const double g11 = 2*e72;
    const double e87 = e59*e76;
    const double g14 = -1.0/20.0*e29;
    const double g16 = -1.0/50.0*e17*e3;
    const double g19 = -e4*m.W;
    const double g23 = -1.0/600.0*e47;
    const double g31 = -1.0/600.0*e51;
    const double g32 = -1.0/600.0*e52;
    const double g34 = -1.0/800000.0*e56;
    const double g37 = (1.0/40.0)*e13*e34*m.U*m.mu;
    const double g43 = (1.0/30.0)*e19*e61 + (1.0/50.0)*e59*m.K*m.P0;
    const double g50 = 4*sq(e3);
    const double g51 = e4*e59;
    const double g52 = -e72;
    const double g55 = -1.0/320000000.0*e29;
    const double g57 = -e69;
    const double g62 = 10*e29;
    const double g63 = -1.0/12000.0*e29*e65;
    const double g68 = e66*e87 + e87;
    const double g75 = (1.0/6000.0)*e19*e34*e35*m.mu;
    const double g77 = (1.0/8000.0)*e13*e34*e35*m.mu;
    const double g84 = -1.0/1600.0*sq(e56)*e65;
    vz[0][i] = e3;
    vz[1][i] = g3;
    vz[2][i] = g5;
    vz[3][i] = e26;
    vz[4][i] = g8;
    vz[5][i] = e29;
    vz[6][i] = e56;
    vz[7][i] = e69;
    vz[8][i] = g11;
    vz[9][i] = g14;
    vz[10][i] = g16;
    vz[11][i] = g19;
    vz[12][i] = g23;
    vz[13][i] = g31;
    vz[14][i] = g32;
    vz[15][i] = g34;
    vz[16][i] = g37;
    vz[17][i] = g43;
    vz[18][i] = g50;
    vz[19][i] = g51;
    vz[20][i] = g52;
    vz[21][i] = g55;
    vz[22][i] = g57;
    vz[23][i] = g62;
    vz[24][i] = g63;
    vz[25][i] = g68;
    vz[26][i] = g75;
    vz[27][i] = g77;
    vz[28][i] = g84;
  }
  __syncthreads();
  if (x0 + lane >= nx) return;
  const int64_t N = (int64_t)nx * ny * nz;
  const double e17 = m.K*m.U;
  const double e34 = sq(m.K);
  const double e35 = sq(m.U);
  const double e38 = m.U*m.W*m.rho0;
  const double e39 = (3.0/50.0)*e38;
  const double e40 = e35*m.rho0;
  const double e41 = e40*m.K;
  const double e43 = (3.0/10000.0)*e41;
  const double e66 = (1.0/(m.gamma - 1));
  const double e76 = 80000*m.P0;
  const double g12 = e34*m.P0*m.kappa/m.rho0;
  const double g20 = (1.0/200.0)*m.rho0;
  const double g22 = -1.0/600.0*e39;
  const double g25 = -1.0/600.0*e43;
  const double g54 = -1.0/4000000.0*m.W;
  const double g67 = -1.0/1600000000.0*e17;
  const double g69 = (1.0/800000000.0)*m.K*m.U;
  const double g73 = (1.0/1600000000.0)*m.K*m.U;
  const double g0 = vx[0][lane];
  const double g4 = vx[1][lane];
  const double e24 = vx[2][lane];
  const double g6 = vx[3][lane];
  const double e67 = vx[4][lane];
  const double g9 = vx[5][lane];
  const double g13 = vx[6][lane];
  const double g17 = vx[7][lane];
  const double g21 = vx[8][lane];
  const double g26 = vx[9][lane];
  const double g29 = vx[10][lane];
  const double g33 = vx[11][lane];
  const double g38 = vx[12][lane];
  const double g40 = vx[13][lane];
  const double g41 = vx[14][lane];
  const double g42 = vx[15][lane];
  const double g44 = vx[16][lane];
  const double g45 = vx[17][lane];
  const double g46 = vx[18][lane];
  const double g53 = vx[19][lane];
  const double g56 = vx[20][lane];
  const double g58 = vx[21][lane];
  const double g61 = vx[22][lane];
  const double g64 = vx[23][lane];
  const double g65 = vx[24][lane];
  const double g66 = vx[25][lane];
  const double g78 = vx[26][lane];
  const double g79 = vx[27][lane];
  const double g81 = vx[28][lane];
  const double g82 = vx[29][lane];
  const int jz = wave % tz;
  if (z0 + jz >= nz) return;
  const double e3 = vz[0][jz];
  const double g3 = vz[1][jz];
  const double g5 = vz[2][jz];
  const double e26 = vz[3][jz];
  const double g8 = vz[4][jz];
  const double e29 = vz[5][jz];
  const double e56 = vz[6][jz];
  const double e69 = vz[7][jz];
  const double g11 = vz[8][jz];
  const double g14 = vz[9][jz];
  const double g16 = vz[10][jz];
  const double g19 = vz[11][jz];
  const double g23 = vz[12][jz];
  const double g31 = vz[13][jz];
  const double g32 = vz[14][jz];
  const double g34 = vz[15][jz];
  const double g37 = vz[16][jz];
  const double g43 = vz[17][jz];
  const double g50 = vz[18][jz];
  const double g51 = vz[19][jz];
  const double g52 = vz[20][jz];
  const double g55 = vz[21][jz];
  const double g57 = vz[22][jz];
  const double g62 = vz[23][jz];
  const double g63 = vz[24][jz];
  const double g68 = vz[25][jz];
  const double g75 = vz[26][jz];
  const double g77 = vz[27][jz];
  const double g84 = vz[28][jz];
  for (int jy = wave / tz; jy < ty && y0 + jy < ny; jy += 4 / tz) {
    const int64_t n = x0 + lane + (int64_t)nx * (y0 + jy + (int64_t)ny * (z0 + jz));
    const double g1 = vy[0][jy];
    const double g2 = vy[1][jy];
    const double e25 = vy[2][jy];
    const double g7 = vy[3][jy];
    const double e68 = vy[4][jy];
    const double g10 = vy[5][jy];
    const double g15 = vy[6][jy];
    const double g18 = vy[7][jy];
    const double g24 = vy[8][jy];
    const double g27 = vy[9][jy];
    const double g28 = vy[10][jy];
    const double g30 = vy[11][jy];
    const double g35 = vy[12][jy];
    const double g36 = vy[13][jy];
    const double g39 = vy[14][jy];
    const double g47 = vy[15][jy];
    const double g48 = vy[16][jy];
    const double g49 = vy[17][jy];
    const double g59 = vy[18][jy];
    const double g60 = vy[19][jy];
    const double g70 = vy[20][jy];
    const double g71 = vy[21][jy];
    const double g72 = vy[22][jy];
    const double g74 = vy[23][jy];
    const double g76 = vy[24][jy];
    const double g80 = vy[25][jy];
    const double g83 = vy[26][jy];
    const double e12 = g0 + g1;
    const double e16 = g2 + g3;
    const double e22 = g4 + g5;
    const double e27 = g6 + g7 + g8;
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
    const double e75 = g10 + g11 + g9;
    const double e77 = e75*e76;
    const double e78 = e27*e70 + e66*e77 + e77;
    const double e79 = e17*e78;
    const double e80 = (1.0/(e27));
    const double e81 = e75*e80;
    const double e82 = e75*sq(e80);
    const double e83 = e80*g12;
    const double e85 = 2*e44;
    S[0 * N + n] = (float)(g20*(e12*g17 + e16*g15 + e22*g16 + e27*g18 + e28*g13 + e28*g14 + g19));
    S[1 * N + n] = (float)(e12*e16*g24 + e12*e27*g28 + e16*e27*g27 + e22*e37*g25 + e36*g26 + e37*g22 + e46*g21 + e46*g23 + g29 + g30);
    S[2 * N + n] = (float)(e12*e16*g26 + e16*e27*g35 + e16*g31 + e50*g24 + e53*g32 + e54*g23 + e54*g33 + e57*g34 + g36 + g37);
    S[3 * N + n] = (float)(e12*e22*g41 + e22*g31 + e27*g40 + (-1.0/400000.0)*e45*e64 + e46*g38 + e53*g24 + e57*g33 + e57*g39 + e63*g32 + g42 + g43);
    S[4 * N + n] = (float)(e12*g67*(e70*g65 + (-1)*e85*(e12*g61 + e22*g64) + g66) + e12*g76 + e12*g79 + e16*g73*(e70*g71 + e85*(e12*g70 + e16*e68) + g72) + e16*g77 + e16*g80 + e22*e27*g81 + e22*g69*((-5)*e44*(e16*e56 + e64) + (-1)*e71 + g68) + e22*g75 + e22*g78 + e71*g54 + e78*g74 + e79*g53 + e79*g55 + (-5)*e83*(e24*e81 + e80*g45 + e82*g44 + g46) + (-3)*e83*(e25*e81 + e80*g48 + e82*g47 + g49) + (-2)*e83*(e26*e81 + e80*g51 + e82*g50 + g52) + g58*(e68 + g56 + g57) + g60*(e67 + e69 + g59) + g63*(e68 + g61 + g62) + g82 + g83 + g84);
  }
}

// One lane per cell, all of it evaluated there: for lattices whose rows are a fraction of a
// tile's 64 cells (rule and times in lbm_mms_source), and for any size.
__global__ void __launch_bounds__(256) k_mms_source_cells(lbm_mms m, int32_t nx, int32_t ny, int32_t nz, double t,
                                                           float* __restrict__ S) {
  const int64_t N = (int64_t)nx * ny * nz;
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = n / nx;
  const double x = (double)(n - row * nx);
  const double z = (double)(row / ny);
  const double y = (double)(row % ny);
  const double e0 = m.K*z;
  const double e1 = m.W*t;
  const double e2 = e0 + e1;
  double e3, e26;
  sincos(e2, &e3, &e26);
  const double e4 = 4*e3;
  const double e5 = m.K*x;
  double e24, e6;
  sincos(e5, &e24, &e6);
  const double e7 = 200*m.a;
  const double e8 = m.K*y;
  double e9, e25;
  sincos(e8, &e9, &e25);
  const double e10 = e5 + 2.0/5.0;
  double e23, e11;
  sincos(e10, &e23, &e11);
  const double e12 = 7*e11 + e7 + 5*e9;
  double e56, e13;
  sincos(e0, &e56, &e13);
  const double e14 = e8 + 9.0/10.0;
  double e15, e30;
  sincos(e14, &e15, &e30);
  const double e16 = 5*e13 + 7*e15 + e7;
  const double e17 = m.K*m.U;
  const double e18 = e0 + 17.0/10.0;
  double e29, e19;
  sincos(e18, &e29, &e19);
  const double e20 = e1 + e5;
  double e21, e62;
  sincos(e20, &e21, &e62);
  const double e22 = 5*e19 + 3*e21 + e7;
  const double e27 = 5*e24 + 3*e25 + 2*e26 + 100;
  const double e28 = e17*e27;
  const double e31 = e5 + 6.0/5.0;
  double e32, e73;
  sincos(e31, &e32, &e73);
  const double e33 = e32*m.P0;
  const double e34 = sq(m.K);
  const double e35 = sq(m.U);
  const double e36 = sq(e12);
  const double e37 = e12*e3;
  const double e38 = m.U*m.W*m.rho0;
  const double e39 = (3.0/50.0)*e38;
  const double e40 = e35*m.rho0;
  const double e41 = e40*m.K;
  const double e42 = (9.0/20000.0)*e41*e9;
  const double e43 = (3.0/10000.0)*e41;
  const double e44 = e27*e40;
  const double e45 = e44*m.K;
  const double e46 = e12*e45;
  const double e47 = (3.0/4000.0)*e29;
  const double e48 = e1 + e8;
  double e74, e49;
  sincos(e48, &e74, &e49);
  const double e50 = sq(e16);
  const double e51 = e3*e39;
  const double e52 = e3*e43;
  const double e53 = e16*e22;
  const double e54 = e16*e45;
  const double e55 = (21.0/20000.0)*e23;
  const double e57 = e22*e45;
  const double e58 = e0 + 3.0/5.0;
  double e72, e59;
  sincos(e58, &e72, &e59);
  const double e60 = e34*m.mu;
  const double e61 = e60*m.U;
  const double e63 = sq(e22);
  const double e64 = e22*e29;
  const double e65 = e35*e60;
  const double e66 = (1.0/(m.gamma - 1));
  const double e67 = 7*e23;
  const double e68 = 7*e30;
  const double e69 = 5*e29;
  const double e70 = e40*(e36 + e50 + e63);
  const double e71 = e3*e70;
  const double e75 = 2*e72 + 5*e73 + 3*e74 + 100;
  const double e76 = 80000*m.P0;
  const double e77 = e75*e76;
  const double e78 = e27*e70 + e66*e77 + e77;
  const double e79 = e17*e78;
  const double e80 = (1.0/(e27));
  const double e81 = e75*e80;
  const double e82 = e75*sq(e80);
  const double e83 = e34*e80*m.P0*m.kappa/m.rho0;
  const double e84 = 240000*e49*m.P0;
  const double e85 = 2*e44;
  const double e86 = 400000*e33;
  const double e87 = e59*e76;
  S[0 * N + n] = (float)((1.0/200.0)*m.rho0*((1.0/20.0)*e12*e6*m.K*m.U - 3.0/100.0*e16*e17*e9 - 1.0/50.0*e17*e22*e3 - 7.0/100.0*e23*e28 + (7.0/100.0)*e27*e30*m.K*m.U - 1.0/20.0*e28*e29 - e4*m.W));
  S[1 * N + n] = (float)((7.0/150.0)*e11*e34*m.U*m.mu - 1.0/600.0*e12*e16*e42 + (7.0/4000000.0)*e12*e27*e30*e35*m.K*m.rho0 + (1.0/800000.0)*e16*e25*e27*e35*m.K*m.rho0 - 1.0/600.0*e22*e37*e43 - 7.0/2000000.0*e23*e46 - 1.0/20.0*e33*m.K + (1.0/40.0)*e34*e9*m.U*m.mu + (1.0/800000.0)*e35*e36*e6*m.K*m.rho0 - 1.0/600.0*e37*e39 - 1.0/600.0*e46*e47);
  S[2 * N + n] = (float)((1.0/800000.0)*e12*e16*e35*e6*m.K*m.rho0 + (1.0/40.0)*e13*e34*m.U*m.mu + (7.0/150.0)*e15*e34*m.U*m.mu + (7.0/2000000.0)*e16*e27*e30*e35*m.K*m.rho0 - 1.0/600.0*e16*e51 - 1.0/600.0*e42*e50 - 1.0/600.0*e47*e54 + (3.0/100.0)*e49*m.K*m.P0 - 1.0/600.0*e52*e53 - 1.0/600.0*e54*e55 - 1.0/800000.0*e56*e57);
  S[3 * N + n] = (float)((1.0/800000.0)*e12*e22*e41*e6 + (1.0/30.0)*e19*e61 + (3.0/200.0)*e21*e61 - 1.0/600.0*e22*e51 + (3.0/20000.0)*e27*e38*e62 + (7.0/4000000.0)*e30*e57 - 1.0/600.0*e42*e53 - 1.0/400000.0*e45*e64 + (3.0/4000000.0)*e46*e62 - 1.0/600.0*e52*e63 - 1.0/600.0*e55*e57 + (1.0/50.0)*e59*m.K*m.P0);
  S[4 * N + n] = (float)((7.0/30000.0)*e11*e12*e34*e35*m.mu - 1.0/1600000000.0*e12*e17*(-5*e6*e70 + e66*e86 - e85*(-e12*e67 + 3*e22*e62) + e86) + (1.0/8000.0)*e12*e34*e35*e9*m.mu + (1.0/8000.0)*e13*e16*e34*e35*m.mu + (7.0/30000.0)*e15*e16*e34*e35*m.mu + (1.0/1600000000.0)*e16*m.K*m.U*(e66*e84 - 3*e70*e9 + e84 + e85*(5*e12*e25 + e16*e68)) + (1.0/6000.0)*e19*e22*e34*e35*m.mu + (3.0/40000.0)*e21*e22*e34*e35*m.mu + (3.0/4000000.0)*e22*e27*e35*e62*m.W*m.rho0 + (1.0/800000000.0)*e22*m.K*m.U*(-5*e44*(e16*e56 + e64) + e66*e87 - e71 + e87) - 7.0/60000.0*e23*e65*(14*e23 + e68 - e69) - 7.0/1600000000.0*e23*e79 - 1.0/1600.0*sq(e25)*e65 - 1.0/12000.0*e29*e65*(10*e29 - e67 + e68) - 1.0/320000000.0*e29*e79 - 7.0/60000.0*e30*e65*(14*e30 + e67 + e69) + (7.0/1600000000.0)*e30*e78*m.K*m.U + (3.0/100.0)*e49*e66*m.P0*m.W - 1.0/1600.0*sq(e56)*e65 - 9.0/40000.0*sq(e62)*e65 - 1.0/4000000.0*e71*m.W - 5*e83*(e24*e81 + 10*e32*e6*e80 + 10*sq(e6)*e82 - e73) - 3*e83*(e25*e81 + 6*e49*e80*e9 - e74 + 6*e82*sq(e9)) - 2*e83*(e26*e81 + 4*sq(e3)*e82 + e4*e59*e80 - e72));
}

}  // namespace

extern "C" lbm_status lbm_mms_source(const lbm_mms* m, int32_t nx, int32_t ny, int32_t nz, double t,
                                     float* S_dev, void* hip_stream) {
  if (!m || !S_dev) return grlbm::fail(LBM_EINVAL, "constants or source array is NULL");
  if (nx < 1 || ny < 1 || nz < 1) return grlbm::fail(LBM_EINVAL, "empty lattice %d x %d x %d", nx, ny, nz);
  const int64_t N = (int64_t)nx * ny * nz;
  if (N > ((int64_t)1 << 31)) return grlbm::fail(LBM_EINVAL, "%lld cells exceed 2^31", (long long)N);
  // the largest tiles that still give 512 blocks, two for each CU: larger ones share more
  // of the sines and cosines (128^3: 23 us with 16 rows, 25 with 8), smaller ones leave a
  // wave fewer rows to do one after another (24^3: 5.1 us with 8 rows, 6.2 with 16)
  int ty = TY, tz = TZ;
  auto blocks = [&] {
    return (((int64_t)nx + TX - 1) / TX) * (((int64_t)ny + ty - 1) / ty) * (((int64_t)nz + tz - 1) / tz);
  };
  while (blocks() < 512 && (tz > 1 || ty > 8)) (tz > 1 ? tz : ty) /= 2;
  // Beyond one turn of blocks a tile costs the card 3-5 ns for its tables and 0.4-0.6 ns
  // for each wave's row, however few cells the row has, and a cell evaluated by itself 0.031
  // ns, so rows of up to 14 cells, and single rows, are evaluated per cell: 1 x 1024 x 1024
  // cells 38 us (tiles 486, before the tiles 112), 8 x 512 x 512 65 us (148, 220), 3000000
  // x 1 x 1 92 us (269, 313); 16 x 512 x 512 would take 132 us against 120 in tiles, 300 x 5
  // x 300 17 against 12.  A launch holds fewer than 2^24 blocks, and lattices with more
  // tiles, those near 2^31 cells along one axis among them, are evaluated per cell as well.
  const int64_t wave_rows = ((int64_t)nx + TX - 1) / TX * ny * nz;
  if (blocks() > 512 && (blocks() >= (1 << 24) || N < 100 * blocks() + 13 * wave_rows))
    hipLaunchKernelGGL(k_mms_source_cells, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, (hipStream_t)hip_stream, *m,
                       nx, ny, nz, t, S_dev);
  else
    hipLaunchKernelGGL(k_mms_source, dim3((unsigned)blocks()), dim3(256), 0, (hipStream_t)hip_stream, *m, nx, ny, nz,
                       ty, tz, t, S_dev);
  HIP_TRY(hipGetLastError());
  return LBM_OK;
}
