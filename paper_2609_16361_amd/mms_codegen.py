"""Generate csrc/grlbm_mms.hip: the source of the manufactured solution on the GPU.

The manufactured solution of Sec. 3.1 (eq. 8) is an exact solution of eq. 1 once
its source S = dQ/dt + div Phi is added.  This script writes eq. 2 (conserved
state, flux with the Newtonian stress and the Fourier flux at constant mu and
kappa, T = p/rho) and the fields of eq. 8 in SymPy, differentiates symbolically,
eliminates common subexpressions, and prints a HIP kernel that evaluates the five
components of S at every cell of an n^3 lattice in FP64 and stores them as FP32.
What depends on one coordinate alone (all the sines and cosines, terms and factors)
is evaluated once per coordinate of a block's tile and kept in LDS.  A second kernel
evaluates all of it per cell, for lattices that fill the tiles badly.
The constants (rho0, U, P0, a, K, W, gamma, mu, kappa, lattice units) stay
symbolic, so one kernel serves every resolution.

Run:  python -m paper_2609_16361_amd.mms_codegen   (rewrites csrc/grlbm_mms.hip)
"""
import os

import sympy as sp

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "csrc", "grlbm_mms.hip")
CONSTS = ("rho0", "U", "P0", "a", "K", "W", "gamma", "mu", "kappa")


def source_expressions():
    """The five components of S as SymPy expressions of (x, y, z, t) and CONSTS."""
    x, y, z, t = sp.symbols("x y z t", real=True)
    c = {n: sp.Symbol("m_" + n, real=True) for n in CONSTS}
    K, W, U, P0, r0, a = c["K"], c["W"], c["U"], c["P0"], c["rho0"], c["a"]
    g, mu, kap = c["gamma"], c["mu"], c["kappa"]
    R = sp.Rational
    rho = r0 * (1 + R(5, 100) * sp.sin(K * x) + R(3, 100) * sp.cos(K * y) + R(2, 100) * sp.cos(K * z + W * t))
    u = [U * (a + R(35, 1000) * sp.cos(K * x + R(4, 10)) + R(25, 1000) * sp.sin(K * y)),
         U * (a + R(35, 1000) * sp.sin(K * y + R(9, 10)) + R(25, 1000) * sp.cos(K * z)),
         U * (a + R(25, 1000) * sp.cos(K * z + R(17, 10)) + R(15, 1000) * sp.sin(K * x + W * t))]
    p = P0 * (1 + R(5, 100) * sp.cos(K * x + R(12, 10)) + R(3, 100) * sp.sin(K * y + W * t)
              + R(2, 100) * sp.sin(K * z + R(6, 10)))
    X = (x, y, z)
    E = p / (g - 1) + rho * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2) / 2
    T = p / rho
    grad_u = [[sp.diff(u[j], X[k]) for k in range(3)] for j in range(3)]
    div_u = grad_u[0][0] + grad_u[1][1] + grad_u[2][2]
    tau = [[mu * (grad_u[j][k] + grad_u[k][j] - (R(2, 3) * div_u if j == k else 0)) for k in range(3)]
           for j in range(3)]
    q = [-kap * sp.diff(T, X[k]) for k in range(3)]
    Q = [rho, rho * u[0], rho * u[1], rho * u[2], E]
    flux = [[rho * u[k] for k in range(3)]]
    for j in range(3):
        flux.append([rho * u[j] * u[k] + (p if j == k else 0) - tau[j][k] for k in range(3)])
    flux.append([(E + p) * u[k] - (tau[k][0] * u[0] + tau[k][1] * u[1] + tau[k][2] * u[2]) + q[k]
                 for k in range(3)])
    S = [sp.diff(Q[f], t) + sum(sp.diff(flux[f][k], X[k]) for k in range(3)) for f in range(5)]
    return (x, y, z, t), c, S


def ccode(e) -> str:
    # a square as a product: pow() evaluates a logarithm and an exponential
    return sp.ccode(e, user_functions={"Pow": [(lambda b, n: n == 2, lambda b, n: f"sq({b})"),
                                               (lambda b, n: n == -1, lambda b, n: f"(1.0/({b}))")]})


def group_by_coordinate(subs, red, dep, axes):
    """Inside expressions of several coordinates, the terms of a sum and the factors of
    a product that depend on one coordinate become one value of that coordinate, with
    the constants among them, so that a cell's own work is what mixes coordinates.  New
    symbols are entered in dep and defined before use."""
    known, out = {}, []
    names = sp.numbered_symbols("g")

    def of(e):
        return set().union(*(dep[f] for f in e.free_symbols))

    def value(e):
        if e.is_Atom:
            return e
        if e not in known:
            known[e] = next(names)
            dep[known[e]] = of(e)
            out.append((known[e], e))
        return known[e]

    def walk(e):
        if len(of(e)) < 2:
            return value(e)
        if not (e.is_Add or e.is_Mul):
            return e if e.is_Atom else e.func(*(walk(a) for a in e.args))
        fixed = e.func(*(a for a in e.args if not of(a)))
        rest = [walk(a) for a in e.args if len(of(a)) > 1]
        for v in axes:
            part = e.func(*(a for a in e.args if of(a) == {v}))
            if part != e.identity:
                part, fixed = e.func(part, fixed), e.identity
                rest.append(value(part))
        if fixed != e.identity:
            rest.append(value(fixed))
        return e.func(*rest, evaluate=False)

    for s, e in subs:
        out.append((s, walk(e) if len(dep[s]) > 1 else e))
    return out, [walk(e) for e in red]


def generate() -> str:
    axes, c, S = source_expressions()
    t = axes[3]
    axes = axes[:3]
    subs, red = sp.cse(S, symbols=sp.numbered_symbols("e"), optimizations="basic")
    # one division serves a reciprocal and its square
    recip = {e.base: s for s, e in subs if e.is_Pow and e.exp == -1}
    subs = [(s, e.subs({b ** -2: r ** 2 for b, r in recip.items()})) for s, e in subs]
    # the coordinates each subexpression depends on
    dep = {v: {v} for v in axes}
    dep.update({v: set() for v in list(c.values()) + [t]})
    for sym, ex in subs:
        dep[sym] = set().union(*(dep[f] for f in ex.free_symbols))
    per_cell = subs, red
    subs, red = group_by_coordinate(subs, red, dep, axes)
    single = {v: [(s, e) for s, e in subs if dep[s] == {v}] for v in axes}
    common = [(s, e) for s, e in subs if not dep[s]]
    mixed = [(s, e) for s, e in subs if len(dep[s]) > 1]
    # what the cells use of each coordinate's values
    used = set().union(*(e.free_symbols for _, e in mixed), *(e.free_symbols for e in red))
    keep = {v: [s for s, _ in single[v] if s in used] for v in axes}

    def code(pairs, indent):
        # a sine and a cosine of the same argument come from one call
        trig = {(type(e), e.args[0]): s for s, e in pairs if isinstance(e, (sp.sin, sp.cos))}
        lines, done = [], set()
        for s, e in pairs:
            if s in done:
                continue
            sn, cs = (trig.get((f, e.args[0])) if isinstance(e, (sp.sin, sp.cos)) else None for f in (sp.sin, sp.cos))
            if sn and cs:
                lines.append(f"{indent}double {sn}, {cs};\n{indent}sincos({ccode(e.args[0])}, &{sn}, &{cs});")
                done |= {sn, cs}
            else:
                lines.append(f"{indent}const double {s} = {ccode(e)};")
        return "\n".join(lines)

    def needed(pairs, exprs):
        """The pairs that the expressions need, directly or through one another."""
        want = set().union(*(e.free_symbols for e in exprs)) if exprs else set()
        out = []
        for s, e in reversed(pairs):
            if s in want:
                out.append((s, e))
                want |= e.free_symbols
        return out[::-1]

    parts = {}
    for v in axes:
        base = needed(common, [e for _, e in single[v]])
        store = "\n".join(f"    v{v}[{i}][i] = {s};" for i, s in enumerate(keep[v]))
        parts[f"AXIS_{v}"] = "\n".join(x for x in (code(base, "    "), code(single[v], "    "), store) if x)
        parts[f"N{v}"] = str(len(keep[v]))
    parts["COMMON"] = code(needed(common, [e for _, e in mixed] + list(red)), "  ")
    parts["LOADX"] = "\n".join(f"  const double {s} = vx[{i}][lane];" for i, s in enumerate(keep[axes[0]]))
    parts["LOADZ"] = "\n".join(f"  const double {s} = vz[{i}][jz];" for i, s in enumerate(keep[axes[2]]))
    parts["LOADY"] = "\n".join(f"    const double {s} = vy[{i}][jy];" for i, s in enumerate(keep[axes[1]]))
    parts["MIXED"] = code(mixed, "    ")
    parts["OUT"] = "\n".join(f"    S[{f} * N + n] = (float)({ccode(red[f])});" for f in range(5))
    parts["CELL"] = code(per_cell[0], "  ")
    parts["CELLOUT"] = "\n".join(f"  S[{f} * N + n] = (float)({ccode(per_cell[1][f])});" for f in range(5))
    out = TEMPLATE
    for k, body in parts.items():
        for n in CONSTS:
            body = body.replace("m_" + n, "m." + n)
        out = out.replace(f"@{k}@", body)
    return out


TEMPLATE = r'''// grlbm_mms.hip -- GENERATED by paper_2609_16361_amd/mms_codegen.py; do not edit.
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
  __shared__ double vx[@Nx@][TX], vy[@Ny@][TY], vz[@Nz@][TZ];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntx = (nx + TX - 1) / TX, nty = (ny + ty - 1) / ty;
  const int r = (int)(blockIdx.x / ntx);
  const int x0 = (int)(blockIdx.x % ntx) * TX, y0 = (r % nty) * ty, z0 = (r / nty) * tz;
  const int i = lane;
  if (wave == 0) {
    const double x = (double)(x0 + i);
@AXIS_x@
  } else if (wave == 1 && i < ty) {
    const double y = (double)(y0 + i);
@AXIS_y@
  } else if (wave == 2 && i < tz) {
    const double z = (double)(z0 + i);
@AXIS_z@
  }
  __syncthreads();
  if (x0 + lane >= nx) return;
  const int64_t N = (int64_t)nx * ny * nz;
@COMMON@
@LOADX@
  const int jz = wave % tz;
  if (z0 + jz >= nz) return;
@LOADZ@
  for (int jy = wave / tz; jy < ty && y0 + jy < ny; jy += 4 / tz) {
    const int64_t n = x0 + lane + (int64_t)nx * (y0 + jy + (int64_t)ny * (z0 + jz));
@LOADY@
@MIXED@
@OUT@
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
@CELL@
@CELLOUT@
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
'''


if __name__ == "__main__":
    src = generate()
    with open(OUT, "w") as fh:
        fh.write(src)
    print(f"wrote {OUT} ({len(src.splitlines())} lines)")
