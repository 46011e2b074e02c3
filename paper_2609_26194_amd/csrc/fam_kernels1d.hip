// fam_kernels1d.hip - HIP kernels of the 1D FAM step and the per-step
// bookkeeping (time step, clipping, termination) for gfx950.
//
// 1D tile: a block of 64 lanes covers cells i0-1 .. i0+62 (lane t <-> cell i0-1+t)
// and writes cells i0 .. i0+61.  The state of cells i0-2 .. i0+63 is staged in LDS;
// each lane reconstructs its cell (appendix "One-dimensional reconstruction
// coefficients"), publishes its share of either interface's flux, and the Shu-Osher
// update of eq. (3) uses
//   R0 = -(f_{i+1/2} - f_{i-1/2})/dx,
//   R1 = (sum_g w_g f(p(xi_g)) - (f_{i+1/2} + f_{i-1/2})/2)/dx     (eq. 1dSemi).
// OE (Prop. 2.1, eq. 1dOE_system, Table sigma1d): jumps at both interfaces of the
// cell, Type I / II denominator over Lambda_i = {i-1, i, i+1}, sigma = max over
// components, u^(1) <- u^(1) exp(-beta dt sigma / dx).
#include "fam_char.h"
#include "fam_device.h"
#include "fam_kernels.h"

namespace fam {

// lanes per block: one wave, so that a barrier costs nothing and the tiles spread over
// the CUs (4000 cells, k = 5 Euler: stage 4.62 us against 4.92 with 256 lanes and 5.8
// before the faces took shares; the launch itself is about 2.5)
constexpr int T1 = 64;
constexpr int OUT1 = T1 - 2;      // cells written per block

// 1D Gauss nodes in the oracle's order: -GS1, -GS0, GS0, GS1
__device__ __forceinline__ constexpr double g1x(int q) {
  return q == 0 ? -GS1 : q == 1 ? -GS0 : q == 2 ? GS0 : GS1;
}
__device__ __forceinline__ constexpr double g1w(int q) { return (q == 0 || q == 3) ? GW1 : GW0; }

template <int K>
__device__ __forceinline__ double poly1d(const double* c, double x) {
  double v = 0.0;
#pragma unroll
  for (int l = 0; l < K; ++l) v = fma(c[l], leg(l, x), v);
  return v;
}

template <class P>
__device__ __forceinline__ P make_phys1(const PhysParams& pp);
template <>
__device__ __forceinline__ Advection make_phys1<Advection>(const PhysParams& pp) { return Advection{pp.ax, pp.ay}; }
template <>
__device__ __forceinline__ Burgers make_phys1<Burgers>(const PhysParams& pp) { return Burgers{pp.ax, pp.ay}; }
template <>
__device__ __forceinline__ Euler<1> make_phys1<Euler<1>>(const PhysParams& pp) { return Euler<1>(pp.gamma); }

// one stage input in LDS: column x of a plane holds cell i0-2+x, and lane t of the
// block cell i0-1+t (column t+1)
struct Tile1 {
  double* u;    // [NC*2][W]: averages and moments
  double* hi;   // [NC][W]: what lane t gives its right face
  double* lo;   // [NC][W]: and its left face
  int W;
  __device__ __forceinline__ double at(int p, int x) const { return u[p * W + x]; }
};
template <int NC, int T>
struct TileStore1 {
  double u[NC * 2 * (T + 2)], hi[NC * (T + 2)], lo[NC * (T + 2)];
  __device__ __forceinline__ Tile1 tile() { return Tile1{u, hi, lo, T + 2}; }
};

// 1D launches of up to 32 waves keep their maximum in slot 0: there the collisions
// (12 ns each) cost less than the reading of all slots (120 cells, 2 waves: a step
// is 4 % slower with slots; 4000 cells, 63 waves: 3 % faster)
__device__ __forceinline__ bool alpha_spread1(int nx) { return nx > 32 * 64; }

// even and odd parts of a reconstruction at x: p(x) = e + o, p(-x) = e - o
template <int K>
__device__ __forceinline__ void pair1d(const double* c, double x, double& e, double& o) {
  e = c[0];
  o = c[1] * x;
#pragma unroll
  for (int l = 2; l < K; ++l) {
    if (l % 2 == 0) e = fma(c[l], leg(l, x), e);
    else o = fma(c[l], leg(l, x), o);
  }
}

template <int K>
constexpr int nb1d() { return K <= 4 ? (K == 3 ? 3 : 4) : K; }   // coefficients of p

// reconstruction of component c of lane t's cell
template <int K>
__device__ __forceinline__ void recon1(const Tile1& S, int c, int t, double* cf) {
  coeffs1d<K>(S.at(2 * c, t), S.at(2 * c, t + 1), S.at(2 * c, t + 2), S.at(2 * c + 1, t), S.at(2 * c + 1, t + 1),
              S.at(2 * c + 1, t + 2), cf);
}

// Shu-Osher update of lane t's cell (all lanes of the block call): L = u + dt R(u),
// R0 = (fL - fR)/dx, R1 = (sum_g w_g f(p(x_g)) - (fL + fR)/2)/dx.  A cell gives each
// of its faces its share f(trace) +- alpha trace, and the two cells of a face add
// the same two shares, so one barrier suffices and the fluxes cancel exactly.
template <int K, class P, bool CHAR>
__device__ __forceinline__ void stage1_cell(const P& phys, const Tile1& S, int t, double ax, double dtx,
                                            double (&L)[P::NC][2]) {
  constexpr int NC = P::NC, NB = nb1d<K>();
  double cf[NC][6];
  if constexpr (CHAR) {
    // in the characteristic variables of this cell's average (L on the stencil,
    // reconstruction per field, R on the coefficients)
    double La[NC][NC], Ra[NC][NC];
    {
      double a[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) a[c] = S.at(2 * c, t + 1);
      char_basis_x<1>(phys.g, a, La, Ra);
    }
#pragma unroll
    for (int w = 0; w < NC; ++w) {
      double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int o = 0; o < 3; ++o) v[3 * m + o] = fma(La[w][c], S.at(2 * c + m, t + o), v[3 * m + o]);
      coeffs1d<K>(v[0], v[1], v[2], v[3], v[4], v[5], cf[w]);
    }
#pragma unroll
    for (int l = 0; l < NB; ++l) {
      double tw[NC];
#pragma unroll
      for (int w = 0; w < NC; ++w) tw[w] = cf[w][l];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double x = 0.0;
#pragma unroll
        for (int w = 0; w < NC; ++w) x = fma(Ra[c][w], tw[w], x);
        cf[c][l] = x;
      }
    }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) recon1<K>(S, c, t, cf[c]);
  }
  {
    double rt[NC], lt[NC], gr[NC], gl[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double e, o;
      pair1d<NB>(cf[c], 0.5, e, o);
      rt[c] = e + o;
      lt[c] = e - o;
    }
    phys.face(0, rt, ax, gr);
    phys.face(0, lt, -ax, gl);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      S.hi[c * S.W + t] = gr[c];
      S.lo[c * S.W + t] = gl[c];
    }
  }
  double V[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) V[c] = 0.0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    double vp[NC], vm[NC], fp[NC], fm[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double e, o;
      pair1d<NB>(cf[c], q == 0 ? GS0 : GS1, e, o);
      vp[c] = e + o;
      vm[c] = e - o;
    }
    phys.flux(0, vp, fp);
    phys.flux(0, vm, fm);
#pragma unroll
    for (int c = 0; c < NC; ++c) V[c] = fma(q == 0 ? GW0 : GW1, fp[c] + fm[c], V[c]);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double fL = S.hi[c * S.W + (t > 0 ? t - 1 : 0)] + S.lo[c * S.W + t];   // twice the face fluxes
    const double fR = S.hi[c * S.W + t] + S.lo[c * S.W + t + 1];
    L[c][0] = fma(0.5 * dtx, fL - fR, S.at(2 * c, t + 1));
    L[c][1] = fma(dtx, fma(-0.25, fL + fR, V[c]), S.at(2 * c + 1, t + 1));
  }
}

// sigma of lane t's cell (all lanes call); D, eps: the bounds of Type I
template <int K, class P>
__device__ __forceinline__ double oe1_sigma(const Tile1& S, int t, int type, double gamma_k, const double* D1,
                                            const double* eps1) {
  constexpr int NC = P::NC, NB = nb1d<K>();
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    double cf[6], e, o;
    recon1<K>(S, c, t, cf);
    pair1d<NB>(cf, 0.5, e, o);
    S.hi[c * S.W + t] = e + o;
    S.lo[c * S.W + t] = e - o;
  }
  __syncthreads();
  double sig = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double J = fabs(S.lo[c * S.W + t] - S.hi[c * S.W + (t > 0 ? t - 1 : 0)]) +
                     fabs(S.lo[c * S.W + t + 1] - S.hi[c * S.W + t]);
    double D, eps;
    if (type == 2) {
      const double a = S.at(2 * c, t), b = S.at(2 * c, t + 1), d = S.at(2 * c, t + 2);
      const double Ssum = (a + b) + d;
      D = fmax(fmax(fabs(a - Ssum), fabs(b - Ssum)), fabs(d - Ssum));
      eps = 1e-14 * fmax(fmax(fmax(fabs(a), fabs(b)), fabs(d)), 1.0);
    } else {
      D = D1[c];
      eps = eps1[c];
    }
    const double s = (D < eps) ? 0.0 : gamma_k * J / D;
    sig = fmax(sig, s);
  }
  return sig;
}

template <int NC>
__device__ __forceinline__ void load_tile1(const Tile1& S, const double* __restrict__ U, const Inst& in, int i0) {
  for (int x = threadIdx.x; x < S.W; x += blockDim.x) {
    const int gi = ghost(i0 - 2 + x, in.nx, in.bcx);
#pragma unroll
    for (int p = 0; p < NC * 2; ++p) S.u[p * S.W + x] = U[in.offset + p * in.plane + gi];
  }
}

template <int K, class P, bool CHAR = false>
__global__ void __launch_bounds__(T1) stage1d_kernel(StageArgs A, Inst in) {
  constexpr int NC = P::NC;
  __shared__ TileStore1<NC, T1> store;
  if (*A.done) return;
  const Tile1 S = store.tile();
  const P phys = make_phys1<P>(A.phys);
  const int t = threadIdx.x;
  const int i0 = blockIdx.x * OUT1;
  const int i = i0 - 1 + t;
  const double dtx = *in.dt / in.dx;
  load_tile1<NC>(S, A.Us, in, i0);
  double ax, ay;
  if (alpha_spread1(in.nx)) alpha_max(alpha_load(in.alpha_in), ax, ay);
  else ax = in.alpha_in[0];
  __syncthreads();
  double L[NC][2];
  stage1_cell<K, P, CHAR>(phys, S, t, ax, dtx, L);
  double amax = 0.0;
  bool bad = false;
  if (t >= 1 && t <= OUT1 && i < in.nx) {
    double avg[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const size_t idx = in.offset + (c * 2 + m) * in.plane + i;
        const double v = (A.ca == 0.0) ? L[c][m] : fma(A.ca, A.U0[idx] - L[c][m], L[c][m]);
        A.Uout[idx] = v;
        if (m == 0) avg[c] = v;
      }
    }
    amax = phys.speed(0, avg, bad);
  }
  amax = wave_max(amax);
  const bool any_bad = __any(bad);
  if ((t & 63) == 0) {
    const unsigned wave = blockIdx.x * (T1 / 64) + t / 64;
    atomic_max_nonneg(alpha_slot(in.alpha_out, alpha_spread1(in.nx) ? wave : 0), amax);
    if (any_bad) atomicOr(A.flag, 1);
  }
}

template <int K, class P>
__global__ void __launch_bounds__(T1) oe1d_kernel(OEArgs A, Inst in) {
  constexpr int NC = P::NC;
  __shared__ TileStore1<NC, T1> store;
  if (*A.done) return;
  const Tile1 S = store.tile();
  const P phys = make_phys1<P>(A.phys);
  const int t = threadIdx.x;
  const int i0 = blockIdx.x * OUT1;
  const int i = i0 - 1 + t;
  const double dt = *in.dt;
  load_tile1<NC>(S, A.Un, in, i0);
  double D1[NC], eps1[NC];
  if (A.type != 2) {
#pragma unroll
    for (int c = 0; c < NC; ++c) type1_bounds(A.stats, in, c, D1[c], eps1[c]);
  }
  __syncthreads();
  const double sig = oe1_sigma<K, P>(S, t, A.type, A.gamma_k, D1, eps1);
  bool bad = false;
  if (t >= 1 && t <= OUT1 && i < in.nx) {
    double beta = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double avg[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) avg[c] = S.at(2 * c, t + a);
      beta = fmax(beta, phys.speed(0, avg, bad));
    }
    const double delta = exp(-beta * dt * sig / in.dx);
    if (A.delta_out) A.delta_out[i] = delta;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      A.Uout[in.offset + (c * 2) * in.plane + i] = S.at(2 * c, t + 1);
      A.Uout[in.offset + (c * 2 + 1) * in.plane + i] = delta * S.at(2 * c + 1, t + 1);
    }
  }
  if (__any(bad) && (t & 63) == 0) atomicOr(A.flag, 1);
}

template <class P>
__global__ void __launch_bounds__(256) alpha1d_kernel(PhysParams pp, const double* __restrict__ U, Inst in,
                                                      int* flag) {
  const P phys = make_phys1<P>(pp);
  constexpr int NC = P::NC;
  bool bad = false;
  double mx = 0.0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < in.nx; i += gridDim.x * blockDim.x) {
    double avg[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) avg[c] = U[in.offset + (c * 2) * in.plane + i];
    mx = fmax(mx, phys.speed(0, avg, bad));
  }
  mx = wave_max(mx);
  const bool any_bad = __any(bad);
  if ((threadIdx.x & 63) == 0) {
    const unsigned wave = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
    atomic_max_nonneg(alpha_slot(in.alpha_out, alpha_spread1(in.nx) ? wave : 0), mx);
    if (any_bad) atomicOr(flag, 1);
  }
}

// ---------------------------------------------------------------------------
// step bookkeeping
// ---------------------------------------------------------------------------
// A step's time step, clock and termination from the wave speeds of its state
// (t, dt, steps, done: the books); false: the run has ended, nothing is to be done.
__device__ __forceinline__ bool begin_step(const StepState& s, double ax, double ay, double dt_fixed, double t_final,
                                           double& t, double& dt, int& steps, int& done) {
  if (done) {
    dt = 0.0;
    return false;
  }
  if (dt_fixed > 0.0) {
    dt = dt_fixed;
  } else {
    dt = (s.dim == 1) ? s.cfl * s.hx / ax : s.cfl / (ax / s.hx + ay / s.hy);
  }
  double tn = t + dt;
  bool go = true;
  if (t_final > 0.0) {
    if (t >= t_final) {
      go = false;
    } else if (tn >= t_final) {
      dt = t_final - t;
      tn = t_final;
    }
  }
  if (!go || !(dt > 0.0) || !(dt < 1e300)) {
    done = 1;
    dt = 0.0;
    return false;
  }
  t = tn;
  steps += 1;
  return true;
}

// Steps of a small 1D mesh in one workgroup: the state stays in LDS and in its
// cell's lane, a barrier takes the place of a launch, and the wave speeds are
// reduced in LDS.  As a sequence of launches such a step is five of 2 to 5 us, each
// bound by its start and its one memory round trip.  Measured, us a step as
// launches / here: Burgers 120 cells k=5 17.4 / 3.4, Euler 400 cells k=6 23.8 / 10.0.
// A run to an end time tests for non-physical averages after the same steps as the
// larger meshes' (first: after `test` steps, 0: not at all; then run_chunk) and stops
// there; a launch that others follow (more) ends at such a step too.
template <int K, class P, bool CHAR = false>
__global__ void __launch_bounds__(run1d_max(P::NC) + 2) run1d_kernel(PhysParams pp, double* __restrict__ U, Inst in, StepState* st,
                                                     int* flag, int nsteps, int test, int more, int fresh,
                                                     double dt_fixed, double t_final, int oe, double gamma_k) {
  constexpr int NC = P::NC;
  extern __shared__ double lds[];
  __shared__ double red[2][16];   // per wave: maxima of the speeds (and of Type I)
  __shared__ double sum[16];      // per wave: Type I sums
  const P phys = make_phys1<P>(pp);
  const int t = threadIdx.x, T = blockDim.x, nw = T >> 6, wv = t >> 6, n = in.nx;
  const int i = t - 1;
  const Tile1 S{lds, lds + NC * 2 * (T + 2), lds + NC * 3 * (T + 2), T + 2};
  double* sp = lds + NC * 4 * (T + 2);   // speeds of the cells of columns x
  const bool own = i >= 0 && i < n;
  bool bad = test > 0 && *flag != 0;   // raised by an earlier call

  // value v of plane p (or of sp) in this lane's column and the ghost columns that mirror it
  auto put = [&](double* plane, double v) {
    if (!own) return;
    plane[i + 2] = v;
    if (in.bcx == 0) {   // periodic
      if (i >= n - 2) plane[i - (n - 2)] = v;
      if (i < 2) plane[i + n + 2] = v;
    } else {             // transmissive
      if (i == 0) plane[0] = plane[1] = v;
      if (i == n - 1) plane[n + 2] = plane[n + 3] = v;
    }
  };
  // largest speed of the lanes' averages, for the waves to read after a barrier
  auto speeds = [&](const double (&u)[NC][2]) {
    double v = 0.0;
    if (own) {
      double avg[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) avg[c] = u[c][0];
      v = fmax(0.0, phys.speed(0, avg, bad));   // a NaN raises the flag and is no maximum
    }
    put(sp, v);
    v = wave_max(v);
    if ((t & 63) == 0) red[0][wv] = v;
  };
  // as bit patterns, like the atomics of the stage kernels
  auto alpha = [&]() {
    unsigned long long m = 0;
    for (int w = 0; w < nw; ++w) m = max(m, (unsigned long long)__double_as_longlong(red[0][w]));
    return __longlong_as_double((long long)m);
  };

  double u[NC][2] = {}, u0[NC][2];
  for (int x = t; x < S.W * NC * 2; x += T) lds[x] = 1.0;   // unused columns: any finite state
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (own) {
      u[c][0] = U[in.offset + (c * 2) * in.plane + i];
      u[c][1] = U[in.offset + (c * 2 + 1) * in.plane + i];
    }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < NC * 2; ++p) put(S.u + p * S.W, u[p / 2][p % 2]);
  speeds(u);
  __syncthreads();

  const StepState s0 = *st;
  double tm = s0.t, dt = fresh ? 0.0 : s0.dt;
  int steps = fresh ? 0 : s0.steps, done = fresh ? 0 : s0.done;
  const double eps1 = 1e-14;
  int k = 0, next = test > 0 ? min(test, nsteps) : nsteps;   // the step before which the run is tested again
#pragma unroll 1
  for (;;) {
#pragma unroll 1
    for (; k < next; ++k) {
      if (!begin_step(s0, alpha(), 0.0, dt_fixed, t_final, tm, dt, steps, done)) break;
      const double dtx = dt / in.dx;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        u0[c][0] = u[c][0];
        u0[c][1] = u[c][1];
      }
#pragma unroll 1
      for (int s = 0; s < 3; ++s) {
        const double ca = s == 0 ? 0.0 : s == 1 ? 0.75 : 1.0 / 3.0;
        double L[NC][2];
        stage1_cell<K, P, CHAR>(phys, S, t, alpha(), dtx, L);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int m = 0; m < 2; ++m) u[c][m] = s == 0 ? L[c][m] : fma(ca, u0[c][m] - L[c][m], L[c][m]);
        __syncthreads();   // the maxima of this stage's input have been read
#pragma unroll
        for (int p = 0; p < NC * 2; ++p) put(S.u + p * S.W, u[p / 2][p % 2]);
        speeds(u);
        __syncthreads();
      }
      if (oe != 0) {
        double D1[NC] = {}, e1[NC] = {};
        if (oe == 1) {
          // Type I: mean, then max |u - mean| and max |u|, over the block
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const double v = wave_sum(own ? u[c][0] : 0.0);
            if ((t & 63) == 0) sum[wv] = v;
            __syncthreads();
            double mu = 0.0;
            for (int w = 0; w < nw; ++w) mu += sum[w];
            mu /= (double)n;
            const double d = wave_max(own ? fabs(u[c][0] - mu) : 0.0), a = wave_max(own ? fabs(u[c][0]) : 0.0);
            __syncthreads();
            if ((t & 63) == 0) {
              sum[wv] = d;
              red[1][wv] = a;
            }
            __syncthreads();
            double M = 0.0;
            for (int w = 0; w < nw; ++w) {
              D1[c] = fmax(D1[c], sum[w]);
              M = fmax(M, red[1][w]);
            }
            e1[c] = eps1 * fmax(M, 1.0);
            __syncthreads();
          }
        }
        const double sig = oe1_sigma<K, P>(S, t, oe, gamma_k, D1, e1);
        const double beta = fmax(fmax(sp[t], sp[t + 1]), sp[t + 2]);
        const double delta = exp(-beta * dt * sig / in.dx);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          u[c][1] = delta * u[c][1];
          put(S.u + (c * 2 + 1) * S.W, u[c][1]);
        }
        __syncthreads();
      }
    }
    if (done || k == nsteps || __syncthreads_or(bad)) break;
    next += run_chunk(t_final - tm, dt);
    if (next > nsteps) {
      if (more) break;
      next = nsteps;
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (own) {
      U[in.offset + (c * 2) * in.plane + i] = u[c][0];
      U[in.offset + (c * 2 + 1) * in.plane + i] = u[c][1];
    }
  if (__any(bad) && (t & 63) == 0) atomicOr(flag, 1);
  if (t == 0) {
    st->t = tm;
    st->dt = dt;
    st->steps = steps;
    st->done = done;
    if (fresh) {
      st->t_final = t_final;
      st->dt_fixed = dt_fixed;
    }
  }
}

// the slots [s0, s0 + n) of wave-speed maxima back to zero (one wave)
__device__ __forceinline__ void alpha_clear(double* s0, int n) {
  for (int k = threadIdx.x; k < n; k += 64)
    *reinterpret_cast<double2*>(s0 + (size_t)k * ALPHA_STRIDE) = make_double2(0.0, 0.0);
}

// A single mesh: one wave, which reads and clears the slots; lane 0 keeps the books.
// A batch (SPREAD = false): a lane per instance.
template <bool SPREAD>
__global__ void __launch_bounds__(64) step_begin_kernel(StepState* st, int ninst, int parity, double dt_fixed,
                                                        double t_final) {
  const int id = SPREAD ? 0 : blockIdx.x * 64 + threadIdx.x;
  if (id >= ninst) return;
  StepState& s = st[id];
  // sets 1, 2 of this parity and 0 of the other are accumulated by this step's stages
  double* in = s.alpha + alpha_set(SPREAD, 3 * parity);
  double* out[3] = {s.alpha + alpha_set(SPREAD, 3 * parity + 1), s.alpha + alpha_set(SPREAD, 3 * parity + 2),
                    s.alpha + alpha_set(SPREAD, 3 * (1 - parity))};
  double ax, ay;
  if constexpr (SPREAD) {
    alpha_max(alpha_load(in), ax, ay);
    alpha_clear(out[0], 2 * ALPHA_SLOTS);
    alpha_clear(out[2], ALPHA_SLOTS);
    if (threadIdx.x != 0) return;
    // slot 0 holds the maximum for the stage kernels that read no other
    in[0] = ax;
    in[1] = ay;
  } else {
    ax = in[0];
    ay = in[1];
    for (double* o : out) o[0] = o[1] = 0.0;
  }
  double t = s.t, dt;
  int steps = s.steps, done = s.done;
  if (begin_step(s, ax, ay, dt_fixed, t_final, t, dt, steps, done)) {
    s.t = t;
    s.steps = steps;
  }
  s.dt = dt;
  s.done = done;
}

template <bool SPREAD>
__global__ void __launch_bounds__(64) reset_steps_kernel(StepState* st, int ninst, double t_final, double dt_fixed) {
  const int id = SPREAD ? 0 : blockIdx.x * 64 + threadIdx.x;
  if (id >= ninst) return;
  StepState& s = st[id];
  if constexpr (SPREAD) {
    alpha_clear(s.alpha, 6 * ALPHA_SLOTS);
    if (threadIdx.x != 0) return;
  } else {
    for (size_t k = 0; k < alpha_inst(false); ++k) s.alpha[k] = 0.0;
  }
  s.dt = 0.0;
  s.t_final = t_final;
  s.dt_fixed = dt_fixed;
  s.steps = 0;
  s.done = 0;
}

void launch_reset_steps(StepState* st, int ninst, double t_final, double dt_fixed, hipStream_t s) {
  if (ninst == 1)
    hipLaunchKernelGGL(reset_steps_kernel<true>, dim3(1), dim3(64), 0, s, st, 1, t_final, dt_fixed);
  else
    hipLaunchKernelGGL(reset_steps_kernel<false>, dim3((ninst + 63) / 64), dim3(64), 0, s, st, ninst, t_final,
                       dt_fixed);
}

// the context clock: every instance's time set to t (a kernel, not a memset, so a
// captured graph may hold it)
__global__ void set_time_kernel(StepState* st, int ninst, double t) {
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id < ninst) st[id].t = t;
}

void launch_set_time(StepState* st, int ninst, double t, hipStream_t s) {
  hipLaunchKernelGGL(set_time_kernel, dim3((ninst + 63) / 64), dim3(64), 0, s, st, ninst, t);
}

void launch_step_begin(StepState* st, int ninst, int parity, double dt_fixed, double t_final, hipStream_t s) {
  if (ninst == 1)
    hipLaunchKernelGGL(step_begin_kernel<true>, dim3(1), dim3(64), 0, s, st, 1, parity, dt_fixed, t_final);
  else
    hipLaunchKernelGGL(step_begin_kernel<false>, dim3((ninst + 63) / 64), dim3(64), 0, s, st, ninst, parity, dt_fixed,
                       t_final);
}

#define FAM_DISPATCH_K1(K_, BODY)                    \
  switch (K_) {                                      \
    case 3: { constexpr int KK = 3; BODY; } break;   \
    case 4: { constexpr int KK = 4; BODY; } break;   \
    case 5: { constexpr int KK = 5; BODY; } break;   \
    case 6: { constexpr int KK = 6; BODY; } break;   \
    default: break;                                  \
  }
#define FAM_DISPATCH_P1(SYS_, BODY)                  \
  switch (SYS_) {                                    \
    case 0: { using PP = Advection; BODY; } break;   \
    case 1: { using PP = Burgers; BODY; } break;     \
    default: { using PP = Euler<1>; BODY; } break;   \
  }

void launch_stage1d(int k, int sys, const StageArgs& A, const Inst& in, hipStream_t s) {
  const dim3 grid((in.nx + OUT1 - 1) / OUT1);
  if (in.charv && sys == 2 && k == 5) {   // characteristic variables: Euler, FAM5
    hipLaunchKernelGGL((stage1d_kernel<5, Euler<1>, true>), grid, dim3(T1), 0, s, A, in);
    return;
  }
  FAM_DISPATCH_P1(sys, FAM_DISPATCH_K1(k, hipLaunchKernelGGL((stage1d_kernel<KK, PP>), grid, dim3(T1), 0, s, A, in)));
}
// steps of a mesh of up to run1d_max cells; fresh: the first of a run (its books start anew)
void launch_run1d(int k, int sys, const PhysParams& pp, double* U, const Inst& in, StepState* st, int* flag,
                  int nsteps, int test, bool more, bool fresh, double dt_fixed, double t_final, int oe,
                  double gamma_k, hipStream_t s) {
  const int T = (in.nx + 2 + 63) / 64 * 64;
  const int nc = sys == 2 ? 3 : 1;
  const size_t lds = sizeof(double) * (nc * 4 + 1) * (T + 2);
  if (in.charv && sys == 2 && k == 5) {
    hipLaunchKernelGGL((run1d_kernel<5, Euler<1>, true>), dim3(1), dim3(T), lds, s, pp, U, in, st, flag, nsteps,
                       test, (int)more, (int)fresh, dt_fixed, t_final, oe, gamma_k);
    return;
  }
  FAM_DISPATCH_P1(sys, FAM_DISPATCH_K1(k, hipLaunchKernelGGL((run1d_kernel<KK, PP>), dim3(1), dim3(T), lds, s, pp, U, in,
                                                            st, flag, nsteps, test, (int)more, (int)fresh, dt_fixed,
                                                            t_final, oe, gamma_k)));
}
void launch_oe1d(int k, int sys, const OEArgs& A, const Inst& in, hipStream_t s) {
  const dim3 grid((in.nx + OUT1 - 1) / OUT1);
  FAM_DISPATCH_P1(sys, FAM_DISPATCH_K1(k, hipLaunchKernelGGL((oe1d_kernel<KK, PP>), grid, dim3(T1), 0, s, A, in)));
}
void launch_alpha1d(int sys, const PhysParams& pp, const double* U, const Inst& in, int* flag, hipStream_t s) {
  const int nb = std::max(1, std::min(256, (in.nx + 255) / 256));
  FAM_DISPATCH_P1(sys, hipLaunchKernelGGL((alpha1d_kernel<PP>), dim3(nb), dim3(256), 0, s, pp, U, in, flag));
}

}  // namespace fam
