// fam_eval.h - point evaluation of the 2D reconstruction and compile-time linear
// functionals of the 3x3 stencil, shared by the forward and adjoint kernels.
#pragma once

#include <utility>

#include "fam_device.h"

namespace fam {

// Gauss node q = 0..3 at -GS1, -GS0, +GS0, +GS1
__device__ __forceinline__ constexpr int qnode(int q) { return (q == 0 || q == 3) ? 1 : 0; }
__device__ __forceinline__ constexpr double qsign(int q) { return q < 2 ? -1.0 : 1.0; }
__device__ __forceinline__ constexpr double qw(int q) { return (q == 0 || q == 3) ? GW1 : GW0; }
__device__ __forceinline__ constexpr double qx(int q) {
  return q == 0 ? -GS1 : q == 1 ? -GS0 : q == 2 ? GS0 : GS1;
}

// index of the basis function L_a(xi) L_b(eta) among those of complete degree k - 1
__host__ __device__ constexpr int basis_index(int a, int b) {
  for (int l = 0; l < 23; ++l)
    if (AX[l] == a && AY[l] == b) return l;
  return -1;
}

// the polynomial in xi that p_k is on the line eta = sy * node(gy) (node 2 = 1/2):
// Q[m] is its coefficient of L_m.  The odd terms come first, so that the compiler
// finds nothing to keep for the opposite line.
template <int K>
__device__ __forceinline__ void line_y(const double* c, int gy, double sy, double* Q) {
#pragma unroll
  for (int m = 0; m < K; ++m) {
    Q[m] = c[basis_index(m, 0)];
#pragma unroll
    for (int b = 1; b + m < K; ++b) Q[m] = fma(c[basis_index(m, b)], (b & 1) ? sy * legn(b, gy) : legn(b, gy), Q[m]);
  }
}

// its values at xi = +X and -X, X = node(gx): one even and one odd part,
// L_3(X) = X (X^2 - 3/20), L_5(X) likewise, so X enters with the last operation
template <int MD>
__device__ __forceinline__ void pair_x(const double* Q, int gx, double& vp, double& vm) {
  const double X = legn(1, gx);
  double ev = fma(Q[2], legn(2, gx), Q[0]), od = Q[1];
  if constexpr (MD >= 4) ev = fma(Q[4], legn(4, gx), ev);
  if constexpr (MD >= 3) od = fma(Q[3], legn(3, gx) / X, od);
  if constexpr (MD >= 5) od = fma(Q[5], legn(5, gx) / X, od);
  vp = fma(X, od, ev);
  vm = fma(-X, od, ev);
}

// Stencil slots that the reconstruction reads: slot 0..8 the averages of the
// 3x3 patch, 9..17 its x-moments, 18..26 its y-moments (patch index b*3 + a).
// For k = 3, 4 only the centre cell's moments enter; for k = 5, 6 the x-moments
// of the cells above and below and the y-moments of the cells left and right
// are not part of the stencil.
template <int K>
__host__ __device__ constexpr bool slot_used(int in) {
  const int l = in % 9;
  if (in < 9) return true;
  if (in < 18) return K >= 5 ? (l != 1 && l != 7) : (l == 4);
  return K >= 5 ? (l != 3 && l != 5) : (l == 4);
}

// ---------------------------------------------------------------------------
// Face-centre values p(1/2, 0), p(-1/2, 0), p(0, 1/2), p(0, -1/2) as linear
// functionals of the stencil inputs u0[1..9], u1[1..9], u2[1..9] (27 slots),
// evaluated at compile time from the coefficient formulas.
// ---------------------------------------------------------------------------
struct CentreWeights {
  double w[4][27];   // [r, l, t, b][u0 1..9, u1 1..9, u2 1..9]
};

template <int K, bool FULL>
__host__ __device__ constexpr CentreWeights make_centre_weights() {
  CentreWeights cw{};
  const double px[4] = {0.5, -0.5, 0.0, 0.0}, py[4] = {0.0, 0.0, 0.5, -0.5};
  const int ncf = FULL ? 23 : ncoef2d(K);
  for (int in = 0; in < 27; ++in) {
    if (!slot_used<K>(in)) continue;
    double u[27] = {};
    u[in] = 1.0;
    double c[23] = {};
    coeffs2d<K>(u, u + 9, u + 18, c, FULL);
    for (int f = 0; f < 4; ++f) {
      double v = 0.0;
      for (int l = 0; l < ncf; ++l) v += c[l] * leg(AX[l], px[f]) * leg(AY[l], py[f]);
      cw.w[f][in] = v;
    }
  }
  return cw;
}

template <int K, bool FULL>
struct CentreTable {
  static constexpr CentreWeights t = make_centre_weights<K, FULL>();
};

// v += w * u[I] with w a compile-time constant (skipped when zero)
template <int K, bool FULL, int F, int I>
__device__ __forceinline__ void centre_acc(double& v, const double (&u)[27]) {
  constexpr double w = CentreTable<K, FULL>::t.w[F][I];
  if constexpr (w != 0.0) v = fma(w, u[I], v);
}

template <int K, bool FULL, int F, int... I>
__device__ __forceinline__ double centre_dot(const double (&u)[27], std::integer_sequence<int, I...>) {
  double v = 0.0;
  (centre_acc<K, FULL, F, I>(v, u), ...);
  return v;
}

// The four values as even and odd parts, p(+-1/2, 0) = ex +- ox, p(0, +-1/2) = ey +- oy,
// over sums of the stencil that share their parity: with the nine values of a plane
// numbered from the lower left, c the centre, xs/xd the right plus/minus the left,
// ys/yd the top and bottom likewise and ss, sd (odd in y), ds (odd in x), dd the corner
// sums.  A weight of such a sum is the signed mean of its members' weights, which differ
// by rounding only; 28 products replace 92.
enum ParitySum { PS_C, PS_XS, PS_XD, PS_YS, PS_YD, PS_SS, PS_SD, PS_DS, PS_DD };
template <int K, bool FULL>
struct ParityWeights {
  double w[4][3][9];   // ex, ox, ey, oy x plane x sum
};
template <int K, bool FULL>
__host__ __device__ constexpr ParityWeights<K, FULL> make_parity_weights() {
  constexpr CentreWeights cw = make_centre_weights<K, FULL>();
  // members (sign by stencil position) of the sums
  const int sg[9][9] = {{0, 0, 0, 0, 1, 0, 0, 0, 0},  {0, 0, 0, 1, 0, 1, 0, 0, 0},  {0, 0, 0, -1, 0, 1, 0, 0, 0},
                        {0, 1, 0, 0, 0, 0, 0, 1, 0},  {0, -1, 0, 0, 0, 0, 0, 1, 0}, {1, 0, 1, 0, 0, 0, 1, 0, 1},
                        {-1, 0, -1, 0, 0, 0, 1, 0, 1}, {-1, 0, 1, 0, 0, 0, -1, 0, 1}, {1, 0, -1, 0, 0, 0, -1, 0, 1}};
  const int xodd[9] = {0, 0, 1, 0, 0, 0, 0, 1, 1}, yodd[9] = {0, 0, 0, 0, 1, 0, 1, 0, 1};
  ParityWeights<K, FULL> r{};
  for (int f = 0; f < 4; ++f)
    for (int m = 0; m < 3; ++m)
      for (int q = 0; q < 9; ++q) {
        // parity of the functional against that of the sum, the moment's own included
        const int px = (xodd[q] + (m == 1)) % 2, py = (yodd[q] + (m == 2)) % 2;
        if (px != (f == 1) || py != (f == 3)) continue;
        double v = 0.0;
        int n = 0;
        for (int l = 0; l < 9; ++l)
          if (sg[q][l] != 0) {
            const int in = m * 9 + l, b = f < 2 ? 0 : 2;
            const double half = f % 2 == 0 ? 0.5 * (cw.w[b][in] + cw.w[b + 1][in]) : 0.5 * (cw.w[b][in] - cw.w[b + 1][in]);
            v += sg[q][l] * half;
            ++n;
          }
        r.w[f][m][q] = v / n;
      }
  return r;
}
template <int K, bool FULL>
struct ParityTable {
  static constexpr ParityWeights<K, FULL> t = make_parity_weights<K, FULL>();
};

// v += w s with w a compile-time constant (skipped when it vanishes to rounding)
template <int K, bool FULL, int F, int M, int Q>
__device__ __forceinline__ void parity_acc(double& v, double s) {
  constexpr double w = ParityTable<K, FULL>::t.w[F][M][Q];
  if constexpr (w > 1e-15 || w < -1e-15) v = fma(w, s, v);
}
template <int K, bool FULL, int F, int M>
__device__ __forceinline__ void parity_plane(double& v, const double (&s)[9]) {
  parity_acc<K, FULL, F, M, 0>(v, s[0]);
  parity_acc<K, FULL, F, M, 1>(v, s[1]);
  parity_acc<K, FULL, F, M, 2>(v, s[2]);
  parity_acc<K, FULL, F, M, 3>(v, s[3]);
  parity_acc<K, FULL, F, M, 4>(v, s[4]);
  parity_acc<K, FULL, F, M, 5>(v, s[5]);
  parity_acc<K, FULL, F, M, 6>(v, s[6]);
  parity_acc<K, FULL, F, M, 7>(v, s[7]);
  parity_acc<K, FULL, F, M, 8>(v, s[8]);
}
__device__ __forceinline__ void parity_sums9(const double (&u)[9], double (&s)[9]) {
  const double t = u[8] + u[6], td = u[8] - u[6], b = u[2] + u[0], bd = u[2] - u[0];
  s[PS_C] = u[4];
  s[PS_XS] = u[5] + u[3];
  s[PS_XD] = u[5] - u[3];
  s[PS_YS] = u[7] + u[1];
  s[PS_YD] = u[7] - u[1];
  s[PS_SS] = t + b;
  s[PS_SD] = t - b;
  s[PS_DS] = td + bd;
  s[PS_DD] = td - bd;
}

// ---------------------------------------------------------------------------
// Transposed reconstruction: RT[in][l] = d c_l / d u_in for the 27 stencil slots
// ---------------------------------------------------------------------------
template <int K>
struct ReconT {
  double w[27][23];
};

template <int K>
__host__ __device__ constexpr ReconT<K> make_recon_t() {
  ReconT<K> r{};
  for (int in = 0; in < 27; ++in) {
    if (!slot_used<K>(in)) continue;
    double u[27] = {};
    u[in] = 1.0;
    double c[23] = {};
    coeffs2d<K>(u, u + 9, u + 18, c, false);
    for (int l = 0; l < 23; ++l) r.w[in][l] = c[l];
  }
  return r;
}

template <int K>
struct ReconTable {
  static constexpr ReconT<K> t = make_recon_t<K>();
};

// acc += sum_l RT[IN][l] a[l] over the p_k coefficients (zeros skipped at compile time)
template <int K, int IN, int L>
__device__ __forceinline__ void rt_acc1(double& acc, const double* a) {
  constexpr double w = ReconTable<K>::t.w[IN][L];
  if constexpr (w != 0.0) acc = fma(w, a[L], acc);
}
template <int K, int IN, int... L>
__device__ __forceinline__ double rt_dot(const double* a, std::integer_sequence<int, L...>) {
  double acc = 0.0;
  (rt_acc1<K, IN, L>(acc, a), ...);
  return acc;
}

// acc += sum_f CW[f][IN] b[f] (transposed face-centre functionals)
template <int K, bool FULL, int IN, int F>
__device__ __forceinline__ void cwt_acc1(double& acc, const double* b) {
  constexpr double w = CentreTable<K, FULL>::t.w[F][IN];
  if constexpr (w != 0.0) acc = fma(w, b[F], acc);
}
template <int K, bool FULL, int IN>
__device__ __forceinline__ double cwt_dot(const double* b) {
  double acc = 0.0;
  cwt_acc1<K, FULL, IN, 0>(acc, b);
  cwt_acc1<K, FULL, IN, 1>(acc, b);
  cwt_acc1<K, FULL, IN, 2>(acc, b);
  cwt_acc1<K, FULL, IN, 3>(acc, b);
  return acc;
}


// ---------------------------------------------------------------------------
// Sign-symmetric point groups.  The 32 flux points of a cell form 8 groups of
// 4 points (sx X, sy Y), sx, sy = +-1, with (X, Y) one of (1/2, GS0), (1/2, GS1)
// (x-faces), (GS0, 1/2), (GS1, 1/2) (y-faces) and {GS0, GS1}^2 (volume).
// phi_l(sx X, sy Y) = phi_l(X, Y) sx^(ax_l odd) sy^(ay_l odd): the values at the
// four points follow from four parity sums of the coefficients, and the
// transposed evaluation from four signed sums.  Node indices: 0 = GS0,
// 1 = GS1, 2 = 1/2.  Point s of a group: 0 (+,+), 1 (+,-), 2 (-,+), 3 (-,-).
// ---------------------------------------------------------------------------
template <int L>
__device__ __forceinline__ constexpr int parity_class() {
  return (AX[L] & 1) + 2 * (AY[L] & 1);
}

template <int L, int NXI, int NYI>
__device__ __forceinline__ constexpr double phi_node() {
  return legn(AX[L], NXI) * legn(AY[L], NYI);
}

template <int NXI, int NYI, int... L>
__device__ __forceinline__ void parity_sums(const double* cf, double (&P)[4], std::integer_sequence<int, L...>) {
  P[0] = P[1] = P[2] = P[3] = 0.0;
  ((P[parity_class<L>()] = fma(cf[L], phi_node<L, NXI, NYI>(), P[parity_class<L>()])), ...);
}

template <int NXI, int NYI, int... L>
__device__ __forceinline__ void parity_scatter(double* ab, const double (&Q)[4], double w,
                                               std::integer_sequence<int, L...>) {
  ((ab[L] = fma(w * phi_node<L, NXI, NYI>(), Q[parity_class<L>()], ab[L])), ...);
}

// point s of a group: s = 0 (+,+), 1 (+,-), 2 (-,+), 3 (-,-)
__device__ __forceinline__ constexpr double grp_sx(int s) { return s < 2 ? 1.0 : -1.0; }
__device__ __forceinline__ constexpr double grp_sy(int s) { return (s & 1) ? -1.0 : 1.0; }

template <int NXI, int NYI, int NCF>
__device__ __forceinline__ void group_values(const double* cf, double (&v)[4]) {
  double P[4];
  parity_sums<NXI, NYI>(cf, P, std::make_integer_sequence<int, NCF>{});
  const double a = P[0] + P[1], b = P[0] - P[1], c = P[2] + P[3], d = P[2] - P[3];
  v[0] = a + c;
  v[1] = a - c;
  v[2] = b + d;
  v[3] = b - d;
}

}  // namespace fam
