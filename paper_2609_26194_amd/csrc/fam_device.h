// fam_device.h - device building blocks of the FAM step on gfx950.
//
// * Reconstruction coefficients: the closed-form solutions of the moment
//   systems, written out from the paper's appendices ("One-dimensional
//   reconstruction coefficients"; "Orthogonal basis functions and polynomial
//   coefficients for the 2D reconstruction").  Coefficients are in the local
//   orthogonal basis built from the scaled Legendre polynomials L0..L5 on
//   [-1/2, 1/2]; the 2D basis function phi^(l) is L_{ax[l]}(xi) L_{ay[l]}(eta).
// * Point evaluation at the 4-point Gauss-Legendre nodes exploits the parity of
//   L_m: values at +s and -s come from one even and one odd partial sum.
// * Physics: linear advection, Burgers, Euler (ideal gas).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fam_kernels.h"

namespace fam {

// XCD-aware tile order.  The hardware hands consecutive workgroups to the chip's
// 8 XCDs in turn; tile xcd_tile(L, N) of workgroup L gives each XCD one
// contiguous range of the N tiles (row-major: neighbouring tiles of the same
// rows), so the cache lines that neighbouring tiles share stay in one L2.
// A bijection of [0, N) for any N; only where tiles run changes.
constexpr int NXCD = 8;
__device__ __forceinline__ int xcd_tile(int L, int N) {
  const int x = L % NXCD, slot = L / NXCD, q = N / NXCD, r = N % NXCD;
  return x * q + min(x, r) + slot;
}

// ---------------------------------------------------------------------------
// 4-point Gauss-Legendre rule on [-1/2, 1/2] (nodes +-GS0, +-GS1; weights sum
// to one).  Standard tabulated values of the rule on [-1, 1], halved.
// ---------------------------------------------------------------------------
constexpr double GS0 = 0.16999052179242813240;   // inner node
constexpr double GS1 = 0.43056815579702628761;   // outer node
constexpr double GW0 = 0.32607257743127307131;   // inner weight
constexpr double GW1 = 0.17392742256872692868;   // outer weight

// scaled Legendre polynomials of the paper's orthogonal bases
__host__ __device__ constexpr double leg(int m, double t) {
  return m == 0 ? 1.0
       : m == 1 ? t
       : m == 2 ? t * t - 1.0 / 12.0
       : m == 3 ? t * t * t - 3.0 / 20.0 * t
       : m == 4 ? t * t * t * t - 3.0 / 14.0 * t * t + 3.0 / 560.0
       :          t * t * t * t * t - 5.0 / 18.0 * t * t * t + 5.0 / 336.0 * t;
}

// node value L_m(s) for s in {GS0, GS1, 1/2}: index 0, 1, 2
__host__ __device__ constexpr double legn(int m, int which) {
  return leg(m, which == 0 ? GS0 : which == 1 ? GS1 : 0.5);
}

// 2D basis degrees (x-degree, y-degree) of phi^(0..22)
constexpr int AX[23] = {0, 1, 0, 2, 1, 0, 3, 2, 1, 0, 2, 4, 3, 1, 0, 5, 4, 3, 2, 1, 0, 4, 2};
constexpr int AY[23] = {0, 0, 1, 0, 1, 2, 0, 1, 2, 3, 2, 0, 1, 3, 4, 0, 1, 2, 3, 4, 5, 2, 4};

// number of basis terms of p_k (complete degree k-1): 6, 10, 15, 21
__host__ __device__ constexpr int ncoef2d(int k) { return k * (k + 1) / 2; }
__host__ __device__ constexpr int maxdeg(int k) { return k - 1; }

// ---------------------------------------------------------------------------
// 2D coefficients.  Patch cells 1..9 stored at index l-1 (row-major from
// (i-1, j-1)).  u0: averages (9); u1: x-moments; u2: y-moments (9 each, only
// the entries used by the system are read).  NCQ coefficients are produced:
// 11 (k = 3, 4: Q_4) or 23 (k = 5, 6: Q_6); callers keep the ones they need.
// ---------------------------------------------------------------------------
template <int K>
__host__ __device__ constexpr inline void coeffs2d(const double* u0, const double* u1, const double* u2,
                                                   double* c, bool full) {
  // indices 0..8 = patch cells I_1..I_9
  const double a1 = u0[0], a2 = u0[1], a3 = u0[2], a4 = u0[3], a5 = u0[4], a6 = u0[5],
               a7 = u0[6], a8 = u0[7], a9 = u0[8];
  if constexpr (K <= 4) {
    c[0] = a5;
    c[1] = 12.0 * u1[4];
    c[2] = 12.0 * u2[4];
    c[3] = 0.5 * (a4 - 2.0 * a5 + a6);
    c[4] = 0.25 * (a1 - a3 - a7 + a9);
    c[5] = 0.5 * (a2 - 2.0 * a5 + a8);
    if constexpr (K == 4) {
      c[6] = (5.0 / 11.0) * (a6 - a4) - (120.0 / 11.0) * u1[4];
      c[7] = 0.25 * (-a1 + 2.0 * a2 - a3 + a7 - 2.0 * a8 + a9);
      c[8] = 0.25 * (-a1 + a3 + 2.0 * a4 - 2.0 * a6 - a7 + a9);
      c[9] = (5.0 / 11.0) * (a8 - a2) - (120.0 / 11.0) * u2[4];
    }
  } else {
    const double b1 = u1[0], b3 = u1[2], b4 = u1[3], b5 = u1[4], b6 = u1[5], b7 = u1[6],
                 b9 = u1[8];
    const double e1 = u2[0], e2 = u2[1], e3 = u2[2], e5 = u2[4], e7 = u2[6], e8 = u2[7],
                 e9 = u2[8];
    // sums, differences and second differences along each patch row (L below, 0
    // the cell's own, U above), shared by all coefficients: 74 operations for the
    // 15 coefficients of k = 5 instead of 112 with every formula written out
    const double sL = a1 + a3, dL = a3 - a1, d0 = a6 - a4, sU = a7 + a9, dU = a9 - a7;
    const double qL = sL - 2.0 * a2, q0 = (a4 + a6) - 2.0 * a5, qU = sU - 2.0 * a8;
    const double dyy = (a2 + a8) - 2.0 * a5, cross = dU - dL;
    const double qd = qU - qL, dd = (dL + dU) - 2.0 * d0;
    const double sbL = b1 + b3, dbL = b3 - b1, sb0 = b4 + b6, db0 = b6 - b4, sbU = b7 + b9, dbU = b9 - b7;
    const double sbd = sbL - sbU, dbd = dbL - dbU, sbb = (sbL + sbU) - 2.0 * sb0, dbb = (dbL + dbU) - 2.0 * db0;
    const double qeL = (e1 + e3) - 2.0 * e2, deL = e3 - e1, qeU = (e7 + e9) - 2.0 * e8, deU = e9 - e7;
    const double qes = qeL + qeU, qed = qeL - qeU, des = deL + deU, ded = deL - deU, e0d = e2 - e8, e0s = e2 + e8;
    c[0] = a5;
    c[1] = 12.0 * b5;
    c[2] = 12.0 * e5;
    c[3] = (73.0 / 56.0) * q0 - (135.0 / 28.0) * db0;
    c[4] = (41.0 / 76.0) * cross + (33.0 / 19.0) * (sbd - des);
    c[5] = (73.0 / 56.0) * dyy + (135.0 / 28.0) * e0d;
    c[6] = (595.0 / 324.0) * d0 - (985.0 / 162.0) * sb0 - (2585.0 / 81.0) * b5;
    c[7] = (1695.0 / 2128.0) * qd + (135.0 / 56.0) * dbd - (33.0 / 19.0) * qes;
    c[8] = (1695.0 / 2128.0) * dd - (33.0 / 19.0) * sbb + (135.0 / 56.0) * ded;
    c[9] = (595.0 / 324.0) * (a8 - a2) - (985.0 / 162.0) * e0s - (2585.0 / 81.0) * e5;
    const double lap2 = (qL + qU) - 2.0 * q0;
    c[10] = (59.0 / 56.0) * lap2 + (135.0 / 56.0) * (qed - dbb);
    c[11] = (15.0 / 4.0) * db0 - (5.0 / 8.0) * q0;
    c[12] = -(5.0 / 38.0) * cross - (30.0 / 19.0) * sbd;
    c[13] = (30.0 / 19.0) * des - (5.0 / 38.0) * cross;
    c[14] = -(5.0 / 8.0) * dyy - (15.0 / 4.0) * e0d;
    if (K == 6 || full) {
      c[15] = (77.0 / 18.0) * sb0 + (133.0 / 9.0) * b5 - (35.0 / 36.0) * d0;
      c[16] = -(5.0 / 16.0) * qd - (15.0 / 8.0) * dbd;
      c[17] = (30.0 / 19.0) * sbb - (5.0 / 38.0) * dd;
      c[18] = (30.0 / 19.0) * qes - (5.0 / 38.0) * qd;
      c[19] = -(5.0 / 16.0) * dd - (15.0 / 8.0) * ded;
      c[20] = (35.0 / 36.0) * (a2 - a8) + (77.0 / 18.0) * e0s + (133.0 / 9.0) * e5;
    }
    if (full) {
      c[21] = (15.0 / 8.0) * dbb - (5.0 / 16.0) * lap2;
      c[22] = -(5.0 / 16.0) * lap2 - (15.0 / 8.0) * qed;
    }
  }
}

// ---------------------------------------------------------------------------
// 1D coefficients (appendix "One-dimensional reconstruction coefficients").
// u0m, u00, u0p: averages of cells i-1, i, i+1; u1*: first moments.
// ---------------------------------------------------------------------------
template <int K>
__device__ __forceinline__ void coeffs1d(double u0m, double u00, double u0p, double u1m, double u10,
                                         double u1p, double* c) {
  c[0] = u00;
  c[1] = 12.0 * u10;
  if constexpr (K <= 4) {
    c[2] = 0.5 * (u0m - 2.0 * u00 + u0p);
    if constexpr (K == 4) c[3] = (5.0 / 11.0) * (u0p - u0m) - (120.0 / 11.0) * u10;
  } else {
    const double d2 = u0m - 2.0 * u00 + u0p;
    c[2] = (73.0 / 56.0) * d2 + (135.0 / 28.0) * (u1m - u1p);
    c[3] = (595.0 / 324.0) * (u0p - u0m) - (985.0 / 162.0) * (u1m + u1p) - (2585.0 / 81.0) * u10;
    c[4] = -(5.0 / 8.0) * d2 - (15.0 / 4.0) * (u1m - u1p);
    if constexpr (K == 6)
      c[5] = (35.0 / 36.0) * (u0m - u0p) + (77.0 / 18.0) * (u1m + u1p) + (133.0 / 9.0) * u10;
  }
}

// 1/x from the hardware reciprocal estimate r (relative error at most 4.6e-8) and
// the remainder e = 1 - x r: 1/x = r / (1 - e) = r + r (e + e^2) up to r e^3, below
// 1e-22 of it, so the result is within rounding of 1/x (not IEEE division)
__device__ __forceinline__ double rcp(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// a value that the compiler computes here, for all active lanes: it would move a
// division that only some lanes' selects use into a branch of its own
__device__ __forceinline__ double here(double x) {
  asm volatile("" : "+v"(x));
  return x;
}

// a value that is the same in every lane, moved to scalar registers
__device__ __forceinline__ double uniform(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                          __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// ---------------------------------------------------------------------------
// Physics
// ---------------------------------------------------------------------------
//
// flux: f_d(u).  The 2D stage kernel takes a face flux apart into the shares of its
// two sides, F = 1/2 (f(u-) + alpha u-) + 1/2 (f(u+) - alpha u+): face() is one
// side's f_d(u) + a u with a = +-alpha (the 1/2 is applied to the residual).
// volume() adds a point of weight w to the sums of the volume quadrature and
// volume_sums() turns them into V1, V2, the averages of f_1, f_2; the means of
// the components themselves are the average (the 4 x 4 rule is exact for p_k).
struct Advection {
  static constexpr int NC = 1;
  double ax, ay;
  struct Volume {};
  __device__ __forceinline__ void face(int d, const double* u, double a, double* g) const {
    g[0] = ((d == 0 ? ax : ay) + a) * u[0];
  }
  __device__ __forceinline__ void volume(const double*, double, Volume&) const {}
  __device__ __forceinline__ void volume_sums(const double* mean, const Volume&, double* V1, double* V2) const {
    V1[0] = ax * mean[0];
    V2[0] = ay * mean[0];
  }
  __device__ __forceinline__ void flux(int d, const double* u, double* f) const {
    f[0] = (d == 0 ? ax : ay) * u[0];
  }
  __device__ __forceinline__ double speed(int d, const double* u, bool& bad) const {
    bad |= !(u[0] == u[0]);
    return fabs(d == 0 ? ax : ay);
  }
};

struct Burgers {
  static constexpr int NC = 1;
  double ax, ay;
  struct Volume {
    double s;
  };
  __device__ __forceinline__ void face(int, const double* u, double a, double* g) const {
    g[0] = fma(0.5, u[0], a) * u[0];
  }
  __device__ __forceinline__ void volume(const double* u, double w, Volume& V) const { V.s = fma(w * u[0], u[0], V.s); }
  __device__ __forceinline__ void volume_sums(const double*, const Volume& V, double* V1, double* V2) const {
    V1[0] = V2[0] = 0.5 * V.s;
  }
  __device__ __forceinline__ void flux(int, const double* u, double* f) const {
    f[0] = 0.5 * u[0] * u[0];
  }
  __device__ __forceinline__ double speed(int, const double* u, bool& bad) const {
    bad |= !(u[0] == u[0]);
    return fabs(u[0]);
  }
};

// Euler in DIM dimensions: u = (rho, rho u [, rho v], E)
template <int DIM>
struct Euler {
  static constexpr int NC = DIM + 2;
  double g, g1, kh;   // gamma, gamma - 1, -(gamma - 1)/(2 gamma), in scalar registers
  __device__ __forceinline__ explicit Euler(double gamma)
      : g(gamma), g1(uniform(gamma - 1.0)), kh(uniform(-0.5 * (gamma - 1.0) / gamma)) {}
  __device__ __forceinline__ double pressure(const double* u, double inv_rho) const {
    double ke = u[1] * u[1];
    if constexpr (DIM == 2) ke += u[2] * u[2];
    return g1 * (u[NC - 1] - 0.5 * ke * inv_rho);
  }
  __device__ __forceinline__ void flux(int d, const double* u, double* f) const {
    const double inv = rcp(u[0]);
    const double p = pressure(u, inv);
    const double vel = u[1 + d] * inv;
    f[0] = u[1 + d];
    f[1] = u[1] * vel;
    if constexpr (DIM == 2) f[2] = u[2] * vel;
    f[1 + d] += p;
    f[NC - 1] = (u[NC - 1] + p) * vel;
  }
  // sums over the volume points of u_x^2 rho, u_y^2 rho, u_x u_y rho and
  // (E + p) u_x, (E + p) u_y divided by gamma
  struct Volume {
    double xx, yy, xy, hx, hy;
  };
  __device__ __forceinline__ void face(int d, const double* u, double a, double* o) const {
    const double inv = rcp(u[0]);
    double ke = u[1] * u[1];
    if constexpr (DIM == 2) ke = fma(u[2], u[2], ke);
    const double p = g1 * fma(-0.5, ke * inv, u[NC - 1]);
    const double vel = u[1 + d] * inv, va = vel + a;
    o[0] = fma(a, u[0], u[1 + d]);
    o[1 + d] = fma(u[1 + d], va, p);
    if constexpr (DIM == 2) o[2 - d] = u[2 - d] * va;
    o[NC - 1] = fma(u[NC - 1], va, p * vel);
  }
  __device__ __forceinline__ void volume(const double* u, double w, Volume& V) const {
    const double inv = rcp(u[0]);
    const double ke = fma(u[2], u[2], u[1] * u[1]);
    const double h = fma(kh, ke * inv, u[3]);   // (E + p) / gamma
    const double wi = w * inv;
    const double vx = u[1] * wi, vy = u[2] * wi;
    V.xx = fma(u[1], vx, V.xx);
    V.xy = fma(u[1], vy, V.xy);
    V.yy = fma(u[2], vy, V.yy);
    V.hx = fma(h, vx, V.hx);
    V.hy = fma(h, vy, V.hy);
  }
  __device__ __forceinline__ void volume_sums(const double* mean, const Volume& V, double* V1, double* V2) const {
    const double p = g1 * fma(-0.5, V.xx + V.yy, mean[3]);
    V1[0] = mean[1];
    V1[1] = V.xx + p;
    V1[2] = V.xy;
    V1[3] = g * V.hx;
    V2[0] = mean[2];
    V2[1] = V.xy;
    V2[2] = V.yy + p;
    V2[3] = g * V.hy;
  }
  // spectral radius |u_d| + c at a cell average; flags rho <= 0, p <= 0, NaN
  __device__ __forceinline__ double speed(int d, const double* u, bool& bad) const {
    const double inv = rcp(u[0]);
    const double p = pressure(u, inv);
    bad |= !(u[0] > 0.0) || !(p > 0.0);
    return fabs(u[1 + d] * inv) + sqrt(g * p * inv);
  }
};

// ---------------------------------------------------------------------------
// reductions
// ---------------------------------------------------------------------------
// v of the lane that a DPP control pairs with this one within its row of 16
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long v) {
  const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)v, CTRL, 0xf, 0xf, false);
  const unsigned hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), CTRL, 0xf, 0xf, false);
  return (unsigned long long)hi << 32 | lo;
}
// v of a fixed lane, in scalar registers
__device__ __forceinline__ unsigned long long lane64(unsigned long long v, int lane) {
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return (unsigned long long)hi << 32 | lo;
}
// op over the rows of 16 lanes (every lane holds its row's result): lanes 1 and 2
// apart by quad permutes, then the mirrored half row and the mirrored row
template <class F>
__device__ __forceinline__ unsigned long long row_reduce(unsigned long long v, F op) {
  v = op(v, dpp64<0xB1>(v));    // quad_perm [1,0,3,2]
  v = op(v, dpp64<0x4E>(v));    // quad_perm [2,3,0,1]
  v = op(v, dpp64<0x141>(v));   // row_half_mirror
  return op(v, dpp64<0x140>(v));   // row_mirror
}

__device__ __forceinline__ double wave_max(double v) {
  auto op = [](unsigned long long a, unsigned long long b) {
    return (unsigned long long)__double_as_longlong(
        fmax(__longlong_as_double((long long)a), __longlong_as_double((long long)b)));
  };
  const unsigned long long r = row_reduce((unsigned long long)__double_as_longlong(v), op);
  return __longlong_as_double(
      (long long)op(op(lane64(r, 0), lane64(r, 16)), op(lane64(r, 32), lane64(r, 48))));
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// max of non-negative doubles through their bit patterns (order-preserving)
__device__ __forceinline__ void atomic_max_nonneg(double* addr, double v) {
  atomicMax(reinterpret_cast<unsigned long long*>(addr), (unsigned long long)__double_as_longlong(v));
}

// The wave speeds of a state: the largest of its slots (as bit patterns, like the
// atomics), one slot per lane, lanes 32 to 63 the same again.
__device__ __forceinline__ double2 alpha_load(const double* __restrict__ set) {
  return *reinterpret_cast<const double2*>(set + (threadIdx.x & (ALPHA_SLOTS - 1)) * ALPHA_STRIDE);
}
__device__ __forceinline__ void alpha_max(double2 a, double& ax, double& ay) {
  static_assert(ALPHA_SLOTS == 32, "two rows of 16 lanes");
  auto op = [](unsigned long long p, unsigned long long q) { return p > q ? p : q; };
  const unsigned long long x = row_reduce((unsigned long long)__double_as_longlong(a.x), op);
  const unsigned long long y = row_reduce((unsigned long long)__double_as_longlong(a.y), op);
  ax = __longlong_as_double((long long)op(lane64(x, 0), lane64(x, 16)));
  ay = __longlong_as_double((long long)op(lane64(y, 0), lane64(y, 16)));
}
// a wave's slot: one lane adds the wave's maxima
__device__ __forceinline__ double* alpha_slot(double* set, unsigned wave) {
  return set + (wave & (ALPHA_SLOTS - 1)) * ALPHA_STRIDE;
}

// Type I: D_Omega and eps_Omega of component c from the blocks' maxima (every lane)
__device__ __forceinline__ void type1_bounds(const double2* __restrict__ stats, const Inst& in, int c, double& D,
                                             double& eps) {
  const int nb = type1_blocks((size_t)in.nx * in.ny);
  double d = 0.0, a = 0.0;
  for (int b = threadIdx.x & 63; b < nb; b += 64) {
    const double2 v = stats[b * 4 + c];
    d = fmax(d, v.x);
    a = fmax(a, v.y);
  }
  D = wave_max(d);
  eps = 1e-14 * fmax(wave_max(a), 1.0);
}

// ghost-cell index map: periodic wrap or transmissive clamp
__device__ __forceinline__ int ghost(int i, int n, int bc) {
  if (bc == 0) {
    i += i < 0 ? n : i >= n ? -n : 0;
    if (__any((unsigned)i >= (unsigned)n)) {   // beyond one period (a strip wider than the mesh)
      i %= n;
      i += i < 0 ? n : 0;
    }
    return i;
  }
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

}  // namespace fam
