// fam_tiles2d.h - HIP kernels of the 2D FAM step for gfx950.
//
// Work decomposition ("marching strips").  One 64-lane wavefront owns a strip of
// columns: lane l holds column i = i0 - 2 + l.  Lanes 2..61 produce output (60
// columns); lanes 1 and 62 are ring columns whose traces feed the strip's two
// boundary faces; lanes 0 and 63 only load.  The wave marches upwards over the
// rows j0-1 .. j0+H (the first and last are ring rows), keeping a rolling window
// of three state rows (12 planes x 64 columns) in LDS.  Every face flux is evaluated
// exactly once per strip:
//   x-faces: a lane's share of its right face's flux, 1/2 (f(u) + alpha u), is
//            passed to the right neighbour lane by a cross-lane shift, and the
//            resulting face flux is passed back;
//   y-faces: a row's share of its top face's flux is kept for the next row.
// The residual of a cell is complete one row later (after its top face), when
// the Shu-Osher update writes the stage result.
//
// Stage s (eq. 12): Uout = a U0 + b (Us + dt R(Us)), R of eq. (11):
//   R0 = -(Fb_{i+1/2} - Fb_{i-1/2})/dx - (Gb_{j+1/2} - Gb_{j-1/2})/dy
//   R1 = V1/dx - (Fb_{i+1/2} + Fb_{i-1/2})/(2dx) - (Gt_{j+1/2} - Gt_{j-1/2})/dy
//   R2 = V2/dy - (Gb_{j+1/2} + Gb_{j-1/2})/(2dy) - (Ft_{i+1/2} - Ft_{i-1/2})/dx
// with Fb = sum_g w_g F(eta_g), Ft = sum_g w_g eta_g F(eta_g) on x-faces (likewise
// Gb, Gt with xi_g on y-faces), V1, V2 the 4x4 Gauss averages of f1, f2, and the
// Lax-Friedrichs flux using one wave speed per direction: the maximum spectral
// radius over the cell averages of Us.  Each stage also max-reduces the wave
// speeds of its output averages for the next stage (and, after the last stage,
// for the next step's time step).
//
// OE (eqs. 2dOE_sol, 2dOE_system, Table sigma2d): per component, face-centre jumps
// of the reconstruction, J^x, J^y, the Type I / Type II denominator over the 3x3
// patch; sigma = max over components; delta = exp(-beta^x dt sigma^x/dx -
// beta^y dt sigma^y/dy); first moments scaled by delta, averages copied.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "fam_char.h"
#include "fam_device.h"
#include "fam_eval.h"
#include "fam_kernels.h"
#include "fam_strip.h"

namespace fam {

#ifndef FAM_OE_WAVES
#define FAM_OE_WAVES 2
#endif
// occupancy targets (waves per SIMD) handed to the register allocator
#define FAM_STAGE_ATTR(K, CHAR) __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(stage_waves(K, P::NC, CHAR))))
#define FAM_OE_ATTR __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(FAM_OE_WAVES)))

// keeps the scheduler from moving work across this point, which bounds the number
// of live values: between the OE kernel's per-component passes and between the
// parts of a stage row (recon of a component, a line of points, a face)
#define FAM_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------------------
// Optional positivity limiter (Euler): the reconstruction p is replaced by
// avg + theta2 (w - avg), w = p with its density scaled by theta1 toward the
// average, theta1 and theta2 the largest values keeping density and pressure
// >= eps = min(1e-13, rho_avg, p(avg)) at all 32 flux points of the cell.
// Both scalings act on the deviation from the average, so they are applied to
// the non-constant coefficients: rho by theta1 theta2, the other components by
// theta2 (the same point values up to rounding).
// ---------------------------------------------------------------------------
// smallest root in (0, 1] of a t^2 + b t + c (c > 0 and value <= 0 at t = 1), else 1
__device__ __forceinline__ double smallest_root_unit(double a, double b, double c) {
  const double disc = fmax(b * b - 4.0 * a * c, 0.0);
  const double sq = sqrt(disc);
  const double q = -0.5 * (b + (b >= 0.0 ? sq : -sq));
  double r1 = here(q / (a == 0.0 ? 1.0 : a));
  r1 = a == 0.0 ? 2.0 : r1;
  double r2 = here(c / (q == 0.0 ? 1.0 : q));
  if (!(r1 > 0.0 && r1 <= 1.0)) r1 = 2.0;
  if (!(r2 > 0.0 && r2 <= 1.0)) r2 = 2.0;
  const double r = fmin(r1, r2);
  return r > 1.0 ? 1.0 : r;
}


// min over the 32 lanes of each half of the wave (DPP within rows of 16, then
// one exchange between the two rows of the half)
template <int CTRL>
__device__ __forceinline__ double dpp_min(double v) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, 0xF, 0xF, false);
  return fmin(v, __hiloint2double(hi, lo));
}

__device__ __forceinline__ double half_wave_min(double v) {
  v = dpp_min<0xB1>(v);    // quad_perm [1,0,3,2]
  v = dpp_min<0x4E>(v);    // quad_perm [2,3,0,1]
  v = dpp_min<0x141>(v);   // row_half_mirror
  v = dpp_min<0x140>(v);   // row_mirror: the row minimum in all 16 lanes
  return fmin(v, __shfl_xor(v, 16, 64));
}

using ScratchDouble = __attribute__((address_space(5))) double;

// The limiter's cheap sufficient test, by every lane on its own cell: the mask of
// the lanes whose cell needs the exact test, and eps.
template <int K, int NCF, class P>
__device__ __forceinline__ unsigned long long pp_cheap_test(const P& phys, const double (&cf)[P::NC][NCF], bool& bad,
                                                            int lane, double& eps) {
  constexpr int NC = P::NC;
  if constexpr (NC != 4) {
    return 0;
  } else {
    const double g = phys.g;
    double avg[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) avg[c] = cf[c][0];
    const double inv = rcp(avg[0]);
    const double pa = phys.pressure(avg, inv);
    const bool adm = (avg[0] > 0.0) && (pa > 0.0);
    bad |= !adm;
    eps = fmin(fmin(avg[0], pa), 1e-13);
    // every basis function is bounded by its value at the cell corner
    // (|L_m| <= L_m(1/2) on [-1/2, 1/2]), which bounds each component's deviation
    // from its average; if density and the pressure lower bound built from those
    // deviations stay above eps (with a rounding margin), no point can violate and
    // the limiter is the identity.
    double dev[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      dev[c] = 0.0;
#pragma unroll
      for (int l = 1; l < NCF; ++l) dev[c] = fma(fabs(cf[c][l]), leg(AX[l], 0.5) * leg(AY[l], 0.5), dev[c]);
    }
    const double rlo = avg[0] - dev[0];
    const double mm = fabs(avg[1]) + dev[1], nn = fabs(avg[2]) + dev[2];
    const double lim = eps + 1e-12 * (avg[0] + dev[0] + fabs(avg[3]) + dev[3]);
    const double plo = (g - 1.0) * (avg[3] - dev[3] - 0.5 * (mm * mm + nn * nn) * rcp(rlo));
    const bool need = adm & (lane >= 1) & (lane <= LANES - 2) & !((rlo > lim) & (plo > lim));
    return __ballot(need);
  }
}

// Between the two, where many cells of a row fail the cheap test (a discontinuity along
// the row): every lane evaluates its own cell's 32 points, and the cells at which density
// and pressure stay clear of eps at all of them, by margins far above the rounding of
// either evaluation, need no exact test (it would find factors of one).  Returns the
// cells that do.  The margins: 1e-10 of the components' size, and a density of at least
// a hundredth of the average, so that velocities stay within sqrt(200 E / rho).
template <int K, int NCF, int MD, class P>
__device__ __forceinline__ unsigned long long pp_points_test(const P& phys, const double (&cf)[P::NC][NCF],
                                                             unsigned long long todo, double eps) {
  constexpr int NC = P::NC;
  if constexpr (NC != 4) {
    return todo;
  } else {
    double size = fabs(cf[0][0]) + fabs(cf[3][0]);
#pragma unroll
    for (int l = 1; l < NCF; ++l)
      size = fma(fabs(cf[0][l]) + fabs(cf[3][l]), leg(AX[l], 0.5) * leg(AY[l], 0.5), size);
    const double lim = fma(1e-10, size, eps), ce = lim * rcp(phys.g1);
    double rmin = cf[0][0], pmin = 1e300;
    auto point = [&](const double (&u)[NC]) {
      rmin = fmin(rmin, u[0]);
      pmin = fmin(pmin, fma(u[0], u[3] - ce, -0.5 * fma(u[1], u[1], u[2] * u[2])));
    };
    // lines of points: the four volume nodes in y with the x-faces, then the y-faces
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      double up[3][NC], um[3][NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double Q[MD + 1];
        line_y<K>(cf[c], q < 4 ? q >> 1 : 2, (q & 1) ? -1.0 : 1.0, Q);
#pragma unroll
        for (int n = 0; n < (q < 4 ? 3 : 2); ++n) pair_x<MD>(Q, n, up[n][c], um[n][c]);
      }
#pragma unroll
      for (int n = 0; n < (q < 4 ? 3 : 2); ++n) {
        point(up[n]);
        point(um[n]);
      }
      FAM_SCHED_FENCE();
    }
    return todo & __ballot(!(rmin > fmax(lim, 0.01 * cf[0][0]) && pmin > 0.0));
  }
}

// The exact test, called by all 64 lanes of the wave for the few cells (near
// discontinuities) that fail the cheap one: each half of the wave takes one of them
// at a time, lane l evaluating flux point l mod 32 of it, so a pair of cells costs
// the wave a few hundred instructions instead of a divergent 32-point loop.  The
// coefficients come from the cell's own lane by ds_bpermute (122 per pair); staged
// in LDS they took 2 KB per wave and the launch 412 us instead of 391 (2048^2, k = 5).
template <int K, int NCF, int MD, class P>
__device__ __forceinline__ void pp_exact(const P& phys, double (&cf)[P::NC][NCF], unsigned long long todo, double eps,
                                         int lane, int& nwork) {
  constexpr int NC = P::NC;
  if constexpr (NC == 4) {
    // the lane number and gamma are hidden from the optimiser here: it would
    // otherwise compute what depends on them alone (phi, masks, addresses) before
    // the row loop and hold its registers through every row
    double g = phys.g;
    asm volatile("" : "+v"(lane), "+v"(g));
    if (lane == 0) nwork += __popcll(todo);
    // this lane's flux point: right face (1/2, eta_g), left face (-1/2, eta_g),
    // top face (xi_g, 1/2), bottom face (xi_g, -1/2), volume (xi_a, eta_b) at
    // 16 + 4 b + a
    const int pt = lane & 31, half = lane >> 5;
    const double nd[4] = {-GS1, -GS0, GS0, GS1};
    double px, py;
    if (pt < 4) { px = 0.5; py = nd[pt]; }
    else if (pt < 8) { px = -0.5; py = nd[pt - 4]; }
    else if (pt < 12) { px = nd[pt - 8]; py = 0.5; }
    else if (pt < 16) { px = nd[pt - 12]; py = -0.5; }
    else { px = nd[(pt - 16) & 3]; py = nd[(pt - 16) >> 2]; }
    double lx[MD + 1], ly[MD + 1];
#pragma unroll
    for (int m = 1; m <= MD; ++m) {
      lx[m] = leg(m, px);
      ly[m] = leg(m, py);
    }
    const double kk = 2.0 / (g - 1.0);
    double th1 = 1.0, th2 = 1.0;
    do {
      // the next two cells (an odd count: both halves take the last one)
      const int la = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int lb = todo ? __ffsll((long long)todo) - 1 : la;
      todo &= todo - 1ull;
      const int src = half ? lb : la;
      double v[NC], a[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        v[c] = 0.0;
#pragma unroll
        for (int b = MD; b >= 0; --b) {
          double x = __shfl(cf[c][basis_index(0, b)], src);
          if (b == 0) a[c] = x;
#pragma unroll
          for (int m = 1; m + b <= MD; ++m) x = fma(__shfl(cf[c][basis_index(m, b)], src), lx[m], x);
          v[c] = b > 0 ? fma(x, ly[b], v[c]) : v[c] + x;
        }
        FAM_SCHED_FENCE();
      }
      const double e = __shfl(eps, src);
      // density: theta1 from the minimum over the 32 points
      const double rmin = half_wave_min(v[0]);
      const double tr = here((a[0] - e) / (a[0] - rmin));
      const double t1 = rmin < e ? tr : 1.0;
      // pressure along avg -> density-limited point value
      const double rho0 = a[0], m0 = a[1], n0 = a[2], E0 = a[3];
      const double w0 = rho0 + t1 * (v[0] - rho0);
      const double w[4] = {w0, v[1], v[2], v[3]};
      const double pw = P(g).pressure(w, rcp(w0));
      double t2 = 1.0;
      if (__any(pw < e)) {   // for all lanes: no divergent code where the registers are full
        const double qc = 2.0 * rho0 * E0 - (m0 * m0 + n0 * n0) - kk * e * rho0;
        const double rd = w0 - rho0, md = w[1] - m0, nd_ = w[2] - n0, Ed = w[3] - E0;
        const double qa = 2.0 * rd * Ed - (md * md + nd_ * nd_);
        const double qb = 2.0 * (rho0 * Ed + rd * E0) - 2.0 * (m0 * md + n0 * nd_) - kk * e * rd;
        const double root = here(smallest_root_unit(qa, qb, qc));
        t2 = pw < e ? root : 1.0;
      }
      t2 = half_wave_min(t2);
      // each half's results (the same in all its lanes) go to its cell's lane
      const double t1b = __shfl(t1, 32), t2b = __shfl(t2, 32);
      const double t1a = __shfl(t1, 0), t2a = __shfl(t2, 0);
      th1 = lane == la ? t1a : lane == lb ? t1b : th1;
      th2 = lane == la ? t2a : lane == lb ? t2b : th2;
    } while (todo);
    if (__any(th1 < 1.0 || th2 < 1.0)) {
      const double t0 = th1 * th2;   // a factor of one changes nothing
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int l = 1; l < NCF; ++l) cf[c][l] *= c == 0 ? t0 : th2;
    }
  }
}

// cost of a row with n cells tested exactly, in rows without any: ROW_TEST +
// ROW_CELL n.  Measured launch times at 2048^2 (k = 5, four-quadrant data), segment
// list cut by it: 391 us; with 1.3 + 0.1 n 430 us, with 1.5 + 0.2 n 402 us.  (Cycles
// read from the clock, as the list was cut before, do not converge with two waves
// on a SIMD: a row's cycles depend on what the other wave does meanwhile, and the
// segments of one launch took from 164 to 657 us.)
constexpr float ROW_TEST = 1.8f, ROW_CELL = 0.15f;
// From POINTS_MIN cells of a row on the point test comes first; it costs about as much
// as the exact test of POINTS_CELLS cells.  Most rows with limiter work hold one or two
// such cells, but a discontinuity along a row fills it, and the wave that has this row
// ends last: four-quadrant data, us per pass without / with the test, 96x80 1944 / 993,
// 256x256 2639 / 1733, 512x512 3998 / 3063, 2048x2048 15561 / 15030, six meshes of 64^2
// to 128^2 2754 / 1247.  The double Mach reflection's and the characteristic variables'
// kernels, whose registers are full, lose 1 % and 9 % on oblique shocks and go without.
constexpr int POINTS_MIN = 6, POINTS_CELLS = 4;

// ---------------------------------------------------------------------------
// Registers and LDS of a stage wave.  What bounds the kernel is the issue of vector
// instructions (2143 per row of 64 cells at k = 5, 1885 of them FP64), so it
// is written for few of them and for a second wave on the SIMD to fill the gaps:
// two waves have 256 registers and 20 KB of LDS each.  The rows of k = 3..5 fit without
// spilling (k = 5: 120 registers of coefficients, 40 carried from row to row), because
// rows go to LDS past the registers and each line's points are used as soon as they are
// evaluated.  (The limiter's point test, which few rows take, spills within itself: one
// value on a single mesh at k = 5, five and seven in a batch at k = 4 and 5; a test
// watches the counts.)  A single spill in the row's second half is expensive: its reload waits
// for the row prefetch issued before it (33 of them made the kernel 1.5x slower).
// k = 6 (168 registers of coefficients) and the characteristic variables run one
// wave per SIMD and use its 40 KB of LDS instead: what a row hands to the next (20
// values per lane) and the row of the step's start wait there, not in registers.
// Stage launch at 2048^2, k = 5, no limiter: 486 us with one wave per SIMD and 3140
// instructions a row (traces of both sides of a face exchanged, written-out
// coefficient formulas), 430 us with this arithmetic, 385-397 us with two waves.
// With the limiter (four-quadrant data): 483 us before, 391 us.
// ---------------------------------------------------------------------------
template <int K, int NC, bool CHAR>
__host__ __device__ constexpr bool rich_lds() { return stage_waves(K, NC, CHAR) == 1; }

template <bool ON, int NPLU>
struct StageU0 {
  alignas(16) double v[NPLU * LANES];    // row of the step's start that the next iteration finishes
};
template <int NPLU>
struct StageU0<false, NPLU> {};
template <bool ON>
struct StageCarry {
  double2 t[4][LANES];                   // [component]: share of the face above, mean and moment
  double2 y[6][LANES];                   // residual without the top face: [component]: m = 0, 1; [4], [5]: m = 2
};
template <>
struct StageCarry<false> {};

// references to a wave's LDS objects.  They are separate variables, so that the
// compiler knows which of them a row on its way to LDS may touch, and waits for it
// at no other's accesses.
template <int K, int NC, bool CHAR>
struct StageShared {
  Window<3 * NC>& W;
  StageCarry<rich_lds<K, NC, CHAR>()>& cy;
  StageU0<rich_lds<K, NC, CHAR>(), 3 * NC>& u0;
  int& nwork;   // cells of this tile that needed the limiter's exact test
};
#define FAM_STAGE_SHARED(K, NC, CHAR)                         \
  __shared__ Window<3 * NC> s_W;                              \
  __shared__ StageCarry<rich_lds<K, NC, CHAR>()> s_cy;        \
  __shared__ StageU0<rich_lds<K, NC, CHAR>(), 3 * NC> s_u0;   \
  __shared__ int s_nwork;                                     \
  StageShared<K, NC, CHAR> S { s_W, s_cy, s_u0, s_nwork }

// ---------------------------------------------------------------------------
// stage tile
// ---------------------------------------------------------------------------
// sums of the share g = f_2(u) + a u over the four points of the face y = sy/2:
// Gb = sum_q w_q g, Gt = sum_q w_q xi_q g
template <int K, int NCF, class P>
__device__ __forceinline__ void yface_sums(const P& phys, const double (&cf)[P::NC][NCF], double sy, double a,
                                           double (&Gb)[P::NC], double (&Gt)[P::NC]) {
  constexpr int NC = P::NC, MD = maxdeg(K);
  double up[2][NC], um[2][NC];   // values at +xi and -xi of the inner and the outer node
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    double Q[MD + 1];
    line_y<K>(cf[c], 2, sy, Q);
    pair_x<MD>(Q, 0, up[0][c], um[0][c]);
    pair_x<MD>(Q, 1, up[1][c], um[1][c]);
    Gb[c] = Gt[c] = 0.0;
  }
  FAM_SCHED_FENCE();
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const double w = n == 0 ? GW0 : GW1, x = n == 0 ? GS0 : GS1;
    double gp[NC], gm[NC];
    phys.face(1, up[n], a, gp);
    phys.face(1, um[n], a, gm);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Gb[c] = fma(w, gp[c] + gm[c], Gb[c]);
      Gt[c] = fma(w * x, gp[c] - gm[c], Gt[c]);
    }
  }
}

// SPREAD: the wave speeds are accumulated over all slots, else in slot 0 alone
template <int K, class P, bool PP, bool DMR = false, bool CHAR = false, bool SPREAD = true>
__device__ void stage_tile(const P& phys, const StageArgs& A, const Inst& in, int i0, int j0, int H,
                           StageShared<K, P::NC, CHAR>& S, double& amax_x, double& amax_y, bool& bad) {
  constexpr int NC = P::NC;
  constexpr int NCF = ncoef2d(K);
  constexpr int MD = maxdeg(K);
  constexpr int NPLU = NC * 3;
  const int lane = threadIdx.x;
  const int i = i0 - 2 + lane;
  const int rend = min(j0 + H, in.ny);          // exclusive end of output rows
  const bool out_lane = lane >= 2 && lane <= LANES - 3 && i < in.nx;
  // ahead of the rows: reduced while these arrive
  double ax, ay;
  double2 slots = {};
  if constexpr (SPREAD) {
    slots = alpha_load(in.alpha_in);
  } else {
    ax = in.alpha_in[0];
    ay = in.alpha_in[1];
  }
  const double dt = *in.dt;
  const double tb = DMR ? *in.t_end - in.t_ofs * dt : 0.0;   // boundary time of this stage
  const double rxy = uniform(in.dy / in.dx);
  const double cdt = uniform(0.5 * dt / in.dy);
  const bool use_u0 = A.ca != 0.0;
  const double* __restrict__ Us = A.Us + in.offset;
  const double* __restrict__ U0 = A.U0 + in.offset;
  double* __restrict__ Uo = A.Uout + in.offset;
  // moment planes of the output, as an element offset from Uout (0: Uout's own)
  const long long mom_off = A.Uout_mom ? elem_offset(A.Uout, A.Uout_mom) : 0;

  Window<NPLU>& W = S.W;
  constexpr bool RICH = rich_lds<K, NC, CHAR>();
  const bool wide = rows_aligned(Us, in, i0), wide0 = rows_aligned(U0, in, i0);
  const int pc = pair_column(in, i0, lane);
  // rows of the double Mach reflection that hold ghost cells are built in registers
  auto plain_row = [&](int r) { return !DMR || (r >= 0 && r < in.ny && i0 >= 2 && i0 + LANES - 2 <= in.nx); };
  auto built_row = [&](int r) {
    double reg[NPLU];
    fetch_row<NPLU, DMR>(Us, in, i0, r, lane, reg, tb);
    store_row<NPLU>(W, slot_of(r), lane, reg);
  };
#pragma unroll 1
  for (int r = j0 - 2; r <= j0; ++r) {
    if (plain_row(r))
      dma_row<NPLU>(Us, in, in.plane, i0, ghost(r, in.ny, in.bcy), lane, &W.at(slot_of(r), 0, 0), wide, pc);
    else
      built_row(r);
  }

  if constexpr (SPREAD) alpha_max(slots, ax, ay);

  // carried from row to row: the share of the row below in the face between the
  // two (T: mean and moment), and that row's residual without its top face (Y)
  double T[2][NC], Y[NC][3];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    T[0][c] = T[1][c] = Y[c][0] = Y[c][1] = Y[c][2] = 0.0;
    if constexpr (RICH) {
      S.cy.t[c][lane] = make_double2(0.0, 0.0);
      S.cy.y[c][lane] = make_double2(0.0, 0.0);
      if (c < 2) S.cy.y[4 + c][lane] = make_double2(0.0, 0.0);
    }
  }
  dma_wait();

  int sl = slot_of(j0 - 2), sm = slot_of(j0 - 1), sh = slot_of(j0);   // slots of the rows r - 1, r, r + 1
  double avg[NC] = {};          // averages that this iteration (or the last) finished

  auto speeds = [&](bool on) {
    bool b = false;
    const double vx = here(phys.speed(0, avg, b)), vy = here(phys.speed(1, avg, b));
    amax_x = on ? fmax(amax_x, vx) : amax_x;
    amax_y = on ? fmax(amax_y, vy) : amax_y;
    bad |= on && b;
  };

  // the rest of a row, from its reconstruction cf on
  auto finish_row = [&](const double (&cf)[NC][NCF], int r, int tested) __attribute__((always_inline)) {
    const bool fin = r - 1 >= j0;   // this iteration finishes row r-1
    const bool ring_lo = (r == j0 - 1), ring_hi = (r == rend);
    // opaque in every iteration, so that no row of plane offsets is kept (and spilled)
    // across the loop: walking from plane to plane costs two scalar additions
    size_t plane = in.plane;
    asm volatile("" : "+s"(plane));

    // bottom face (i, r-1/2): this row's share completes it
    double Gb[NC], Gt[NC];
    yface_sums<K, NCF>(phys, cf, -1.0, -ay, Gb, Gt);
    FAM_SCHED_FENCE();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if constexpr (RICH) {
        const double2 t = S.cy.t[c][lane], y = S.cy.y[c][lane], z = S.cy.y[4 + c / 2][lane];
        T[0][c] = t.x;
        T[1][c] = t.y;
        Y[c][0] = y.x;
        Y[c][1] = y.y;
        Y[c][2] = c % 2 == 0 ? z.x : z.y;
      }
      Gb[c] += T[0][c];
      Gt[c] += T[1][c];
    }

    // finish the row below: its top face is this row's bottom face.  All lanes
    // compute (those without output on the strip's first column); only the stores
    // are masked, so that no register is moved or spilled under a partial mask.
    if (fin) {
      const ptrdiff_t idx = (ptrdiff_t)(r - 1) * in.nx + (i0 - 2);   // lane 0's column
      const double* q0 = U0 + idx;
      double* q = Uo + idx;
      const int ul = out_lane ? lane : 2;
      // at k = 5 two components at a time: their values of the step's start are read
      // together, and no more are in flight than the registers hold (more, and the
      // compiler waits for each to spill it)
      constexpr int CB = K == 5 && NC == 4 && !RICH ? 2 : NC;
#pragma unroll
      for (int cb = 0; cb < NC; cb += CB) {
        double v[CB * 3];
        if (use_u0) {
#pragma unroll
          for (int p = 0; p < CB * 3; ++p) {
            if constexpr (RICH) v[p] = S.u0.v[(cb * 3 + p) * LANES + lane];
            else v[p] = q0[ul];
            q0 += plane;
          }
        }
#pragma unroll
        for (int c = cb; c < cb + CB; ++c) {
          const double D[3] = {Y[c][0] - Gb[c], Y[c][1] - Gt[c], fma(-0.5, Gb[c], Y[c][2])};
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            const double L = fma(cdt, D[m], W.at(sl, c * 3 + m, lane));
            double& x = v[(c - cb) * 3 + m];
            x = use_u0 ? fma(A.ca, x - L, L) : L;
          }
          avg[c] = v[(c - cb) * 3];
        }
        FAM_SCHED_FENCE();
        if (out_lane) {
#pragma unroll
          for (int p = 0; p < CB * 3; ++p) {
            (p % 3 == 0 ? q : q + mom_off)[lane] = v[p];
            q += plane;
          }
        }
        FAM_SCHED_FENCE();
      }
      if constexpr (!RICH) speeds(out_lane);
    }
    if (ring_hi) return;
    // row r + 2 replaces row r - 1, which nothing reads any more
    const bool pre = r + 2 <= rend + 1, dma = plain_row(r + 2);
    dma_reads_done();
    int dl = lane;
    if constexpr (!RICH) asm volatile("" : "+v"(dl));   // its per-lane addresses are not kept between rows
    if (pre && dma) dma_row<NPLU>(Us, in, plane, i0, ghost(r + 2, in.ny, in.bcy), dl, &W.at(sl, 0, 0), wide, pc);
    if constexpr (RICH) {
      if (use_u0 && !ring_lo) dma_row<NPLU>(U0, in, plane, i0, r, lane, S.u0.v, wide0, pc);
    }
    FAM_SCHED_FENCE();

    if (!ring_lo) {
      // the four interior lines y = eta_q: on each, the x-face points (both
      // sides' shares) and four volume points
      double Fb[NC], Ft[NC];     // left face: mean and moment along it
      typename P::Volume V{};
#pragma unroll
      for (int c = 0; c < NC; ++c) Fb[c] = Ft[c] = 0.0;
      // the wave speeds of the row just finished: a long chain of dependent
      // operations, which a lone wave fills with the first line's independent ones
      // (for all lanes, so that no branch keeps them apart)
      if constexpr (RICH) speeds(fin && out_lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double up[3][NC], um[3][NC];   // values at xi = +-GS0, +-GS1, +-1/2
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double Q[MD + 1];
          line_y<K>(cf[c], qnode(q), qsign(q), Q);
#pragma unroll
          for (int n = 0; n < 3; ++n) pair_x<MD>(Q, n, up[n][c], um[n][c]);
        }
        // the left face takes the left neighbour's right share
        double gr[NC], gl[NC];
        phys.face(0, up[2], ax, gr);
        phys.face(0, um[2], -ax, gl);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const double F = from_left(gr[c]) + gl[c];
          Fb[c] = fma(qw(q), F, Fb[c]);
          Ft[c] = fma(qw(q) * qx(q), F, Ft[c]);
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const double w = (n == 0 ? GW0 : GW1) * qw(q);
          phys.volume(up[n], w, V);
          phys.volume(um[n], w, V);
        }
        FAM_SCHED_FENCE();
      }
      // the right face is the right neighbour's left face
      double Lb[NC], Rb[NC], Lt[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double FbR = from_right(Fb[c]), FtR = from_right(Ft[c]);
        Lb[c] = FbR - Fb[c];
        Rb[c] = FbR + Fb[c];
        Lt[c] = FtR - Ft[c];
      }
      double V1[NC], V2[NC];
      {
        double mean[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) mean[c] = cf[c][0];
        phys.volume_sums(mean, V, V1, V2);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        Y[c][0] = fma(-rxy, Lb[c], Gb[c]);
        Y[c][1] = fma(rxy, fma(-0.5, Rb[c], 2.0 * V1[c]), Gt[c]);
        Y[c][2] = fma(-rxy, Lt[c], fma(-0.5, Gb[c], 2.0 * V2[c]));
      }
    }
    FAM_SCHED_FENCE();
    // this row's share of its top face
    yface_sums<K, NCF>(phys, cf, 1.0, ay, T[0], T[1]);
    if constexpr (RICH) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        S.cy.t[c][lane] = make_double2(T[0][c], T[1][c]);
        if (!ring_lo) {
          S.cy.y[c][lane] = make_double2(Y[c][0], Y[c][1]);
          if (c % 2 == 0) S.cy.y[4 + c / 2][lane] = make_double2(Y[c][2], Y[c + 1][2]);
        }
      }
    }

    if constexpr (DMR) {
      if (pre && !dma) built_row(r + 2);
    }
    dma_wait();
    if constexpr (PP) {
      // the iteration reconstructs (and limits) row r: its cost in plain rows, for
      // the next launch's partition (rows of this segment only)
      if (A.row_cost && lane == 0 && r >= j0 && r < rend)
        A.row_cost[(size_t)(i0 / STRIP) * in.ny + r] = tested > 0 ? ROW_TEST + ROW_CELL * tested : 1.0f;
    }
  };

#pragma unroll 1
  for (int r = j0 - 1; r <= rend; ++r) {
    // reconstruction of all components
    double cf[NC][NCF];
    if constexpr (CHAR) {
      // in the characteristic variables of this cell's average: transform the
      // stencil with L, reconstruct each field, map the coefficients back with R
      double La[NC][NC], Ra[NC][NC];
      {
        double a[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) a[c] = W.at(sm, c * 3, lane);
        char_basis_x<2>(phys.g, a, La, Ra);
      }
#pragma unroll
      for (int w = 0; w < NC; ++w) {
        double u0[9], u1[9], u2[9];
#pragma unroll
        for (int l = 0; l < 9; ++l) u0[l] = u1[l] = u2[l] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double g0[9], g1[9], g2[9];
          gather<K>(W, c, lane, sl, sm, sh, g0, g1, g2);
#pragma unroll
          for (int l = 0; l < 9; ++l) {
            u0[l] = fma(La[w][c], g0[l], u0[l]);
            u1[l] = fma(La[w][c], g1[l], u1[l]);
            u2[l] = fma(La[w][c], g2[l], u2[l]);
          }
        }
        double tmp[23];
        coeffs2d<K>(u0, u1, u2, tmp, false);
#pragma unroll
        for (int l = 0; l < NCF; ++l) cf[w][l] = tmp[l];
      }
#pragma unroll
      for (int l = 0; l < NCF; ++l) {
        double t[NC];
#pragma unroll
        for (int w = 0; w < NC; ++w) t[w] = cf[w][l];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double v = 0.0;
#pragma unroll
          for (int w = 0; w < NC; ++w) v = fma(Ra[c][w], t[w], v);
          cf[c][l] = v;
        }
      }
    } else {
      // a lone wave reads the next component's stencil while it works on this one's
      double u0[2][9], u1[2][9], u2[2][9];
      if constexpr (RICH) gather<K>(W, 0, lane, sl, sm, sh, u0[0], u1[0], u2[0]);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if constexpr (!RICH) gather<K>(W, c, lane, sl, sm, sh, u0[c & 1], u1[c & 1], u2[c & 1]);
        else if (c + 1 < NC) gather<K>(W, c + 1, lane, sl, sm, sh, u0[(c + 1) & 1], u1[(c + 1) & 1], u2[(c + 1) & 1]);
        FAM_SCHED_FENCE();
        double tmp[23];
        coeffs2d<K>(u0[c & 1], u1[c & 1], u2[c & 1], tmp, false);
#pragma unroll
        for (int l = 0; l < NCF; ++l) cf[c][l] = tmp[l];
        FAM_SCHED_FENCE();
      }
    }

    if constexpr (PP) {
      // rare: 0.45 % of the cells, in 4.5 % of the rows of the four-quadrant problem
      double eps = 0.0;
      unsigned long long todo = pp_cheap_test<K, NCF>(phys, cf, bad, lane, eps);
      bool pointwise = false;
      auto limit = [&]() __attribute__((always_inline)) {
        if constexpr (!DMR && !CHAR) {
          pointwise = __popcll(todo) >= POINTS_MIN;
          if (pointwise) todo = pp_points_test<K, NCF, MD>(phys, cf, todo, eps);
        }
        if (todo) pp_exact<K, NCF, MD>(phys, cf, todo, eps, lane, S.nwork);
      };
      if (__builtin_expect(todo != 0, 0)) {
        if constexpr (!RICH && K == 5) {
          // what the row carries waits in scratch memory meanwhile: kept in registers,
          // it or some coefficients would be spilled in every row
          double park[5 * NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            park[5 * c] = T[0][c];
            park[5 * c + 1] = T[1][c];
#pragma unroll
            for (int m = 0; m < 3; ++m) park[5 * c + 2 + m] = Y[c][m];
          }
          asm volatile("" : : "v"((ScratchDouble*)park) : "memory");   // keeps it there
          limit();
          asm volatile("" : : "v"((ScratchDouble*)park) : "memory");
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            T[0][c] = park[5 * c];
            T[1][c] = park[5 * c + 1];
#pragma unroll
            for (int m = 0; m < 3; ++m) Y[c][m] = park[5 * c + 2 + m];
          }
        } else {
          limit();
        }
      }
      finish_row(cf, r, (pointwise ? POINTS_CELLS : 0) + __popcll(todo));
    } else {
      finish_row(cf, r, 0);
    }
    {
      const int t = sl;
      sl = sm;
      sm = sh;
      sh = t;
    }
  }
  if constexpr (RICH) speeds(out_lane && rend > j0);   // the last row's
  __syncthreads();
}

// ---------------------------------------------------------------------------
// OE tile.  The four face-centre values of a cell's reconstruction, p(+-1/2, 0)
// and p(0, +-1/2), are fixed linear functionals of its 3x3 stencil moments
// (weights in fam_eval.h, folded at compile time), taken as even and odd parts.
// ---------------------------------------------------------------------------
struct Centre {
  double xr, xl, yt, yb;   // p(1/2, 0), p(-1/2, 0), p(0, 1/2), p(0, -1/2)
  double D, eps;           // Type II: denominator and its threshold
};

// the hardware's maximum and minimum of two values as they come from memory (fmax
// and fmin of such values first canonicalise each of them)
__device__ __forceinline__ double vmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double vmin(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

template <int K, bool FULL>
__device__ __forceinline__ void centre_values(const double (&u0)[9], const double (&u1)[9], const double (&u2)[9],
                                              Centre& o) {
  double s[9];
  double ex = 0.0, ox = 0.0, ey = 0.0, oy = 0.0;
  parity_sums9(u0, s);
  parity_plane<K, FULL, 0, 0>(ex, s);
  parity_plane<K, FULL, 1, 0>(ox, s);
  parity_plane<K, FULL, 2, 0>(ey, s);
  parity_plane<K, FULL, 3, 0>(oy, s);
  {
    // S = sum, M = max, m = min of the 3x3 averages; max |v - S| = max(M - S, S - m)
    // and max |v| = max(|M|, |m|) (rounding is monotone)
    const double S = (s[PS_C] + s[PS_XS]) + (s[PS_YS] + s[PS_SS]);
    const double M = vmax(vmax(vmax(vmax(u0[0], u0[1]), vmax(u0[2], u0[3])), vmax(vmax(u0[4], u0[5]), vmax(u0[6], u0[7]))),
                          u0[8]);
    const double m = vmin(vmin(vmin(vmin(u0[0], u0[1]), vmin(u0[2], u0[3])), vmin(vmin(u0[4], u0[5]), vmin(u0[6], u0[7]))),
                          u0[8]);
    o.D = vmax(M - S, S - m);
    o.eps = 1e-14 * vmax(vmax(-m, M), 1.0);   // max(|M|, |m|) = max(M, -m)
  }
  parity_sums9(u1, s);
  parity_plane<K, FULL, 0, 1>(ex, s);
  parity_plane<K, FULL, 1, 1>(ox, s);
  parity_plane<K, FULL, 2, 1>(ey, s);
  parity_plane<K, FULL, 3, 1>(oy, s);
  parity_sums9(u2, s);
  parity_plane<K, FULL, 0, 2>(ex, s);
  parity_plane<K, FULL, 1, 2>(ox, s);
  parity_plane<K, FULL, 2, 2>(ey, s);
  parity_plane<K, FULL, 3, 2>(oy, s);
  o.xr = ex + ox;
  o.xl = ex - ox;
  o.yt = ey + oy;
  o.yb = ey - oy;
}

// What bounds it: from a million cells instruction issue and the bytes alike (read 12
// planes, write 8, against 789 instructions a row at k = 5, 998 before the even and
// odd parts), on smaller meshes the rows' latency.  k = 5, us a launch before and after:
// 2048x2048 200 / 185 on average over a run and 157 at the least, 1400x1400 103 / 86
// (floors at the copy rate 133 and 62), a batch of 40 meshes 183 / 167.  A row's reads
// of LDS come first; then the row above the next one is loaded into the slot of the row below, past the vector registers, while this row's
// jumps and the factors of the row below are computed.  Where no more waves could run
// for it, a fourth slot takes that row from the start of the iteration on (scalar
// equations, and launches of at most one wave per SIMD; with two per SIMD three slots of
// the Euler equations are what LDS holds).
template <int K, class P, bool FULL, bool DMR, int SLOTS>
__device__ void oe_tile(const P& phys, const OEArgs& A, const Inst& in, int i0, int j0, int H,
                        Window<3 * P::NC, SLOTS>& W, double (&t1s)[8], bool& bad) {
  constexpr int NC = P::NC;
  constexpr int NPLU = NC * 3;
  constexpr bool DEEP = SLOTS == 4;
  const int lane = threadIdx.x;
  const int i = i0 - 2 + lane;
  const int rend = min(j0 + H, in.ny);
  const bool out_lane = lane >= 2 && lane <= LANES - 3 && i < in.nx;
  const bool type2 = A.type == 2;
  const double dt = *in.dt;
  const double tb = DMR ? *in.t_end : 0.0;   // OE: the end of the step
  const double cx = uniform(dt / in.dx), cy = uniform(dt / in.dy);
  // averages from Ua (NULL: Un), moments from Un, as an element offset from Ua
  const double* __restrict__ Ua = (A.Ua ? A.Ua : A.Un) + in.offset;
  const long long moff = A.Ua ? elem_offset(A.Ua, A.Un) : 0;
  double* __restrict__ Uo = A.Uout + in.offset;
  const bool write_avg = !A.avg_in_place;
  const bool wide = rows_aligned(Ua, in, i0) && (moff & 1) == 0;
  const int pc = pair_column(in, i0, lane);

  // Type I: D_Omega (at 0..NC-1) and eps_Omega (at 4..3+NC) per component, read
  // once into LDS (a global load inside the row loop would make the compiler wait
  // there for every load in flight, the prefetched rows included, on either type)
  if (!type2) {
#pragma unroll 1
    for (int c = 0; c < NC; ++c) type1_bounds(A.stats, in, c, t1s[c], t1s[4 + c]);
  }

  auto load_row = [&](int r, int slot) {
    // rows of the double Mach reflection that hold ghost cells are built in registers
    if (!DMR || (r >= 0 && r < in.ny && i0 >= 2 && i0 + LANES - 2 <= in.nx)) {
      int dl = lane, col = pc;
      if constexpr (K >= 6) {   // its column is not kept between rows: the registers are full
        asm volatile("" : "+v"(dl));
        col = pair_column(in, i0, dl);
      }
      dma_row_split<NPLU>(Ua, moff, in, i0, ghost(r, in.ny, in.bcy), dl, &W.at(slot, 0, 0), wide, col);
    } else {
      double reg[NPLU];
      fetch_row<NPLU, DMR>(Ua, in, i0, r, lane, reg, tb, moff);
      store_row<NPLU>(W, slot, lane, reg);
    }
  };
#pragma unroll 1
  for (int q = 0; q < 3; ++q) load_row(j0 - 2 + q, q);
  dma_wait();
  int sl = 0, sm = 1, sh = 2, sn = DEEP ? 3 : 0;   // slots of the rows r - 1, r, r + 1, r + 2

  double prevTop[NC];      // face-centre value at the top of the row below
  double prevJb[NC];       // |jump| at the bottom face of the row below
  double pJx[NC];          // J^x of the row below
  double pD[NC], pEps[NC]; // denominators of the row below
  double pbx = 0.0, pby = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) prevTop[c] = prevJb[c] = pJx[c] = pD[c] = pEps[c] = 0.0;
  // spectral radii of the rows r - 1, r (carried) and r + 1 of the current row r
  double spx[3], spy[3];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    double a1[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) a1[c] = W.at(q == 0 ? sl : sm, c * 3, lane);
    spx[q] = phys.speed(0, a1, bad);
    spy[q] = phys.speed(1, a1, bad);
  }

#pragma unroll 1
  for (int r = j0 - 1; r <= rend; ++r) {
    if constexpr (DEEP) {
      dma_reads_done();   // the reads of row r - 2, whose slot it is
      if (r + 2 <= rend + 1) load_row(r + 2, sn);
      FAM_SCHED_FENCE();
    }
    // the averages of row r + 1 and what row r - 1 writes
    double a1[NC], own[NC][2];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      a1[c] = W.at(sh, c * 3, lane);
      own[c][0] = W.at(sl, c * 3 + 1, lane);
      own[c][1] = W.at(sl, c * 3 + 2, lane);
    }
    const bool fin = r - 1 >= j0;   // this iteration finishes row r - 1
    const ptrdiff_t idx = (ptrdiff_t)(r - 1) * in.nx + i;
    // one pass per component: the face-centre values and denominators of row r, the
    // sigma of row r - 1 (whose top face is this row's bottom face), row r's jumps
    double sx = 0.0, sy = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double u0[9], u1[9], u2[9];
      gather<K>(W, c, lane, sl, sm, sh, u0, u1, u2);
      if (write_avg && fin && out_lane) Uo[c * 3 * in.plane + idx] = u0[1];   // the OE changes no average
      if (c == NC - 1 && !DMR && !DEEP) {
        dma_reads_done();
        if (r + 2 <= rend + 1) load_row(r + 2, sl);
      }
      Centre ctr;
      centre_values<K, FULL>(u0, u1, u2, ctr);
      const double Jb = fabs(ctr.yb - prevTop[c]);
      const double gD = A.gamma_k * rcp(pD[c]);
      const bool on = !(pD[c] < pEps[c]);
      const double qx = here(gD * pJx[c]), qy = here(gD * (prevJb[c] + Jb));
      sx = on ? fmax(sx, qx) : sx;
      sy = on ? fmax(sy, qy) : sy;
      const double jl = ctr.xl - from_left(ctr.xr);
      const double jr = from_right(jl);
      pJx[c] = fabs(jl) + fabs(jr);
      prevJb[c] = Jb;
      prevTop[c] = ctr.yt;
      pD[c] = type2 ? ctr.D : t1s[c];
      pEps[c] = type2 ? ctr.eps : t1s[4 + c];
      FAM_SCHED_FENCE();
    }
    if constexpr (DMR && !DEEP) {   // later than above, where the built rows find registers
      dma_reads_done();
      if (r + 2 <= rend + 1) load_row(r + 2, sl);
      FAM_SCHED_FENCE();
    }

    // finish the row below
    if (fin) {
      const double delta = here(exp(-pbx * cx * sx - pby * cy * sy));
      if (out_lane) {
        if (A.delta_out) A.delta_out[idx] = delta;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          Uo[(c * 3 + 1) * in.plane + idx] = own[c][0] * delta;
          Uo[(c * 3 + 2) * in.plane + idx] = own[c][1] * delta;
        }
      }
    }
    if (r == rend) break;

    // spectral radii of row r + 1 (each cell once; rows r - 1, r carried) and the
    // wave-speed bounds of row r over the 3x3 patch: column maxima, then the neighbours
    spx[2] = phys.speed(0, a1, bad);
    spy[2] = phys.speed(1, a1, bad);
    const double bx = vmax(vmax(spx[0], spx[1]), spx[2]);
    const double by = vmax(vmax(spy[0], spy[1]), spy[2]);
    pbx = vmax(bx, vmax(from_left(bx), from_right(bx)));
    pby = vmax(by, vmax(from_left(by), from_right(by)));
    spx[0] = spx[1];
    spx[1] = spx[2];
    spy[0] = spy[1];
    spy[1] = spy[2];
    {
      const int t = sl;
      sl = sm;
      sm = sh;
      sh = DEEP ? sn : t;
      sn = t;
    }
    dma_wait();
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// what the kernels share
// ---------------------------------------------------------------------------
template <class P>
__device__ __forceinline__ P make_phys(const PhysParams& pp);
template <>
__device__ __forceinline__ Advection make_phys<Advection>(const PhysParams& pp) {
  return Advection{pp.ax, pp.ay};
}
template <>
__device__ __forceinline__ Burgers make_phys<Burgers>(const PhysParams& pp) {
  return Burgers{pp.ax, pp.ay};
}
template <>
__device__ __forceinline__ Euler<2> make_phys<Euler<2>>(const PhysParams& pp) {
  return Euler<2>(pp.gamma);
}

template <bool SPREAD = true>
__device__ __forceinline__ void flush_wave_results(double amax_x, double amax_y, bool bad,
                                                   double* alpha_out, int* flag) {
  amax_x = wave_max(amax_x);
  amax_y = wave_max(amax_y);
  const bool any_bad = __any(bad);
  if (threadIdx.x == 0) {
    if (alpha_out) {
      double* slot = SPREAD ? alpha_slot(alpha_out, blockIdx.x + blockIdx.y * gridDim.x) : alpha_out;
      atomic_max_nonneg(&slot[0], amax_x);
      atomic_max_nonneg(&slot[1], amax_y);
    }
    if (any_bad) atomicOr(flag, 1);
  }
}

// Position in a heavy-first order (nh tiles with limiter work first, then the
// others) that workgroup L of N takes: the heavy tiles in turn over the XCDs,
// the others in the XCD-aware order (each XCD a contiguous range).  A bijection
// of [0, N).
__device__ __forceinline__ int heavy_first_slot(int L, int N, int nh) {
  if (L < nh) return L;
  const int x = L % NXCD;
  int base = 0, first = 0;
  for (int q = 0; q <= x; ++q) {
    const int f = nh + ((q - nh) % NXCD + NXCD) % NXCD;   // first light position on XCD q
    const int cnt = f < N ? (N - 1 - f) / NXCD + 1 : 0;
    if (q < x) base += cnt;
    else first = f;
  }
  return nh + base + (L - first) / NXCD;
}

#define FAM_DISPATCH_K(K_, BODY)         \
  switch (K_) {                          \
    case 3: { constexpr int KK = 3; BODY; } break; \
    case 4: { constexpr int KK = 4; BODY; } break; \
    case 5: { constexpr int KK = 5; BODY; } break; \
    case 6: { constexpr int KK = 6; BODY; } break; \
    default: break;                      \
  }

#define FAM_DISPATCH_P(SYS_, BODY)                          \
  switch (SYS_) {                                           \
    case 0: { using PP = Advection; BODY; } break;          \
    case 1: { using PP = Burgers; BODY; } break;            \
    default: { using PP = Euler<2>; BODY; } break;          \
  }

}  // namespace fam
