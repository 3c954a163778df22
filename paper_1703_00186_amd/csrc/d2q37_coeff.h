// Device code of the coefficient form of the lattice state.
//
// After a collision with the Hermite projection (Sec. 2) the 37 populations
// of a site are fixed by its 15 relaxed Hermite coefficients b_pq, p + q <= 4:
//   f_l = w_l sum_pq b_pq He_p(c_lx) He_q(c_ly) / (p! q!).
// The coefficient form stores those 15 FP64 numbers instead of the 37
// populations (120 instead of 296 bytes per site); a reader rebuilds a
// population from its source site's coefficients with the same operations
// that made the stored populations before, so nothing is rounded in between.
// The adjoint's mu = B^T C^T lambda has the same structure
//   mu_l = sum_pq B_pq He_p(c_lx) He_q(c_ly)
// (times zero for the populations a wall supplied, which no reader asks for)
// and is stored the same way.
//
// Everything here is written with explicit fused multiply-adds and without
// contraction, so that every kernel that computes the same quantity gets the
// same bits: a run that starts from stored populations and one that starts
// from stored coefficients agree exactly.
#pragma once

#include <hip/hip_runtime.h>

#include "d2q37_device.h"

#pragma clang fp contract(off)

namespace d2q37 {

__host__ __device__ constexpr int slot(int p, int q) {
  for (int k = 0; k < NC; ++k)
    if (kCP[k] == p && kCQ[k] == q) return k;
  return -1;
}

// Geometry of a coefficient buffer: no halos.  Column x is cs doubles long:
// seven planes of pairs, [pitch rows][2] (16-byte accesses), then one plane
// of single values (slot 14).
struct CGeom {
  int lx, ly;
  int periodic;     // periodic y (rows wrap), else walls
  int nw;           // waves that cover a column
  unsigned pitch;   // rows of a plane (ly rounded up to 32)
  long long cs;     // NC * pitch
};

// The walls in coefficient space.  A wall row's unknown populations are
// rho_w v_l (Sec. 2: fixed temperature, zero velocity), so they add
// rho_w V_pq, V_pq = sum over the unknown l of v_l H_pq(c_l), to the
// projection of the known ones; rho_w = a_00(known) / sum over the known l of
// v_l.  Rows 0..2 from the bottom, then ly - 3 .. ly - 1.
struct WallTable {
  double v[6][NC];  // V_pq in storage order
  double ivk[6];    // 1 / sum over the known l of v_l
};

// V_pq and sum_known v are quadratic in th = T_wall - 1: their coefficients.
struct WallBasis {
  double v[3][6][NC], known[3][6];
};
constexpr WallBasis make_wall_basis() {
  WallBasis b{};
  for (int i = 0; i < 6; ++i)
    for (int l = 0; l < Q; ++l) {
      const double x2 = c2(l);
      const double v[3] = {W[l], W[l] * 0.5 * (x2 - 2.0),
                           W[l] * 0.125 * (x2 * x2 - 8.0 * x2 + 8.0)};
      // row i < 3 lacks sources below row 0, row ly - 6 + i those above ly - 1
      const bool unknown = i < 3 ? EY[l] > i : -EY[l] > 5 - i;
      for (int n = 0; n < 3; ++n) {
        if (!unknown) b.known[n][i] += v[n];
        for (int k = 0; unknown && k < NC; ++k)
          b.v[n][i][k] += v[n] * he(EX[l], kCP[k]) * he(EY[l], kCQ[k]);
      }
    }
  return b;
}

inline WallTable make_walls(const Phys& p) {
  constexpr WallBasis b = make_wall_basis();
  WallTable t;
  for (int i = 0; i < 6; ++i) {
    const double th = i < 3 ? p.th_bottom : p.th_top;
    t.ivk[i] = 1.0 / (b.known[0][i] + th * (b.known[1][i] + th * b.known[2][i]));
    for (int k = 0; k < NC; ++k)
      t.v[i][k] = b.v[0][i][k] + th * (b.v[1][i][k] + th * b.v[2][i][k]);
  }
  return t;
}

__device__ __forceinline__ bool wall_row(const CGeom& g, int y, int& i) {
  i = y < 3 ? y : y - g.ly + 6;
  return !g.periodic && (y < 3 || y >= g.ly - 3);
}

__device__ __forceinline__ double mad(double c, double x, double y) {
  return __builtin_fma(c, x, y);
}

// largest |e_y| among the hops with e_x = ex
__host__ __device__ constexpr int reach(int ex) {
  return (ex == 3 || ex == -3) ? 1 : (ex == 2 || ex == -2) ? 2 : 3;
}
__host__ __device__ constexpr int label(int ex, int ey) {
  for (int l = 0; l < Q; ++l)
    if (EX[l] == ex && EY[l] == ey) return l;
  return -1;
}

// The two uses of the expansion and its transpose.
//   Forward: f_l = w_l sum b_pq H_pq / (p! q!),  a_pq = sum f_l H_pq
//   Adjoint: mu_l = sum B_pq H_pq,               L_pq = sum w_l lambda_l H_pq
// (the adjoint's 1 / (p! q!) is applied to the finished L_pq).
struct Forward {
  static __host__ __device__ constexpr double up(int e, int n) { return hef(e, n); }
  static __host__ __device__ constexpr double wup(int l) { return W[l]; }
  static __host__ __device__ constexpr double wdown(int) { return 1.0; }
};
struct Adjoint {
  static __host__ __device__ constexpr double up(int e, int n) { return he(e, n); }
  static __host__ __device__ constexpr double wup(int) { return 1.0; }
  static __host__ __device__ constexpr double wdown(int l) { return W[l]; }
};

// P_q = sum_p b_pq He_p(c_x) (/ p!) for the hops with e_x = ex
template <class K, int ex>
__device__ __forceinline__ void column_sums(const double (&b)[NC], double (&P)[5]) {
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    double s = b[slot(0, q)];
#pragma unroll
    for (int p = 1; p + q < 5; ++p) {
      const double h = K::up(ex, p);
      if (h != 0.0) s = mad(h, b[slot(p, q)], s);
    }
    P[q] = s;
  }
}

// populations (ex, 0) and (ex, +-k) from the column sums: the parts even and
// odd in e_y once, their sum and difference
template <class K, int ex>
__device__ __forceinline__ double population0(const double (&P)[5]) {
  constexpr double w = K::wup(label(ex, 0));
  double e = w == 1.0 ? P[0] : w * P[0];
  e = mad(w * K::up(0, 2), P[2], e);
  return mad(w * K::up(0, 4), P[4], e);
}
template <class K, int ex, int k>
__device__ __forceinline__ void populations(const double (&P)[5], double& plus, double& minus) {
  constexpr double w = K::wup(label(ex, k));
  double e = w == 1.0 ? P[0] : w * P[0];
  e = mad(w * K::up(k, 2), P[2], e);
  e = mad(w * K::up(k, 4), P[4], e);
  double o = (w * K::up(k, 1)) * P[1];
  o = mad(w * K::up(k, 3), P[3], o);
  plus = e + o;
  minus = e - o;
}

// One e_x group of a site's arriving populations: (ex, 0) and (ex, +-k).
struct Group {
  double zero, plus[3], minus[3];
};

// s_q += contributions of (ex, +-k)
template <class K, int ex, int k>
__device__ __forceinline__ void project_pairs(const Group& f, double (&s)[5]) {
  constexpr double w = K::wdown(label(ex, k));
  constexpr double w1 = w * he(k, 1), w2 = w * he(k, 2), w3 = w * he(k, 3), w4 = w * he(k, 4);
  const double sum = f.plus[k - 1] + f.minus[k - 1], dif = f.plus[k - 1] - f.minus[k - 1];
  s[0] = w == 1.0 ? s[0] + sum : mad(w, sum, s[0]);
  s[1] = k == 1 ? w1 * dif : mad(w1, dif, s[1]);
  s[2] = mad(w2, sum, s[2]);
  s[3] = k == 1 ? w3 * dif : mad(w3, dif, s[3]);
  s[4] = mad(w4, sum, s[4]);
  if constexpr (k < reach(ex)) project_pairs<K, ex, k + 1>(f, s);
}

// a_pq += contribution of the group; groups arrive with ex = 3 first (which
// starts the sums), then 2, ... -3
template <class K, int ex>
__device__ __forceinline__ void project_group(const Group& f, double (&a)[NC]) {
  constexpr double w = K::wdown(label(ex, 0));
  const double s0 = w == 1.0 ? f.zero : w * f.zero;
  double s[5] = {s0, 0.0, -s0, 0.0, 3.0 * s0};
  project_pairs<K, ex, 1>(f, s);
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    const double h = he(ex, p);
    if (h == 0.0) continue;
#pragma unroll
    for (int q = 0; p + q < 5; ++q) {
      double& t = a[slot(p, q)];
      if (ex == 3)
        t = p == 0 ? s[q] : h * s[q];
      else
        t = p == 0 ? t + s[q] : mad(h, s[q], t);
    }
  }
}

// the populations of one e_x group of a site from its coefficients
template <class K, int ex>
__device__ __forceinline__ void expand_group(const double (&b)[NC], Group& f) {
  double P[5];
  column_sums<K, ex>(b, P);
  f.zero = population0<K, ex>(P);
  populations<K, ex, 1>(P, f.plus[0], f.minus[0]);
  if constexpr (reach(ex) >= 2) populations<K, ex, 2>(P, f.plus[1], f.minus[1]);
  if constexpr (reach(ex) >= 3) populations<K, ex, 3>(P, f.plus[2], f.minus[2]);
}

template <int ex, int k = 1>
__device__ __forceinline__ void to_labels(const Group& f, double (&v)[Q]) {
  constexpr int zero = label(ex, 0), plus = label(ex, k), minus = label(ex, -k);
  v[zero] = f.zero;
  v[plus] = f.plus[k - 1];
  v[minus] = f.minus[k - 1];
  if constexpr (k < reach(ex)) to_labels<ex, k + 1>(f, v);
}
template <int ex, int k = 1>
__device__ __forceinline__ void from_labels(const double (&v)[Q], Group& f) {
  constexpr int zero = label(ex, 0), plus = label(ex, k), minus = label(ex, -k);
  f.zero = v[zero];
  f.plus[k - 1] = v[plus];
  f.minus[k - 1] = v[minus];
  if constexpr (k < reach(ex)) from_labels<ex, k + 1>(v, f);
}

// all 37 populations of a site <-> its coefficients / their projection
template <class K, int ex = 3>
__device__ __forceinline__ void expand_site(const double (&b)[NC], double (&v)[Q]) {
  Group f;
  expand_group<K, ex>(b, f);
  to_labels<ex>(f, v);
  if constexpr (ex > -3) expand_site<K, ex - 1>(b, v);
}
template <class K, int ex = 3>
__device__ __forceinline__ void project_site(const double (&v)[Q], double (&a)[NC]) {
  Group f;
  from_labels<ex>(v, f);
  project_group<K, ex>(f, a);
  if constexpr (ex > -3) project_site<K, ex - 1>(v, a);
}

// The walls: a holds the projection of the known populations.
__device__ __forceinline__ void wall_coeffs(double (&a)[NC], const WallTable& wt, int i) {
  const double rho_w = a[0] * wt.ivk[i];
#pragma unroll
  for (int k = 0; k < NC; ++k) a[k] = mad(rho_w, wt.v[i][k], a[k]);
}

// collide (Eq. (2) moments, forced equilibrium, relaxation): the projection
// a_pq of the arriving populations becomes the coefficients b_pq.  Mass is
// conserved exactly (b_00 = a_00).
__device__ __forceinline__ void collide_coeffs(double (&a)[NC], const Phys& P) {
  const double rho = a[slot(0, 0)], inv = 1.0 / rho;
  const double ux = a[slot(1, 0)] * inv, uy = a[slot(0, 1)] * inv;
  const double th0 = 0.5 * mad(a[slot(2, 0)] + a[slot(0, 2)], inv, -mad(ux, ux, uy * uy));
  const double Ux = ux + P.tau_gx, Uy = uy + P.tau_gy, th = th0 + P.dtheta;
  const double x2 = Ux * Ux, y2 = Uy * Uy, t3 = 3.0 * th, t6 = 6.0 * th, tt = t3 * th;
  const double hx[5] = {1.0, Ux, x2 + th, Ux * (x2 + t3), mad(x2, x2 + t6, tt)};
  const double hy[5] = {1.0, Uy, y2 + th, Uy * (y2 + t3), mad(y2, y2 + t6, tt)};
  const double keep = 1.0 - P.omega, om_rho = P.omega * rho;
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    const double gp = p == 0 ? om_rho : om_rho * hx[p];
#pragma unroll
    for (int q = 0; p + q < 5; ++q) {
      if (p + q == 0) continue;
      double& t = a[slot(p, q)];
      t = q == 0 ? mad(keep, t, gp) : mad(gp, hy[q], keep * t);
    }
  }
}

// Eq. (2) fields of a site from its coefficients.
__device__ __forceinline__ Macro macro_coeffs(double b00, double b10, double b01, double b20,
                                              double b02) {
  Macro m;
  m.rho = b00;
  m.inv_rho = 1.0 / b00;
  m.ux = b10 * m.inv_rho;
  m.uy = b01 * m.inv_rho;
  m.th = 0.5 * mad(b20 + b02, m.inv_rho, -mad(m.ux, m.ux, m.uy * m.uy));
  return m;
}

// B^T C(m)^T in coefficient space: L holds sum_l w_l lambda_l H_pq at the
// site's arriving populations, m = (rho, j_x, j_y, sum |c|^2 f) the
// pre-collision moments; on return L holds the coefficients B_pq of mu, with
// the wall's share of the unknown populations' adjoint (their sum weighted by
// v_l, over sum_known v) added to every known one: a shift of B_00.
__device__ __forceinline__ void adjoint_coeffs(double (&L)[NC], double rho, double jx, double jy,
                                               double e, const Phys& P) {
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const double s = INVFAC[kCP[k]] * INVFAC[kCQ[k]];
    if (s != 1.0) L[k] = s * L[k];
  }
  const double inv = 1.0 / rho;
  const double ux = jx * inv, uy = jy * inv;
  const double u2 = mad(ux, ux, uy * uy);
  const double th = mad(0.5 * e, inv, -1.0) - 0.5 * u2;
  const double Ux = ux + P.tau_gx, Uy = uy + P.tau_gy, ths = th + P.dtheta;
  // h_n, dh_n/dU, dh_n/dTh of both directions
  const double x2 = Ux * Ux, y2 = Uy * Uy, t3 = 3.0 * ths, tt = t3 * ths;
  const double hx[5] = {1.0, Ux, x2 + ths, Ux * (x2 + t3), mad(x2, mad(6.0, ths, x2), tt)};
  const double hy[5] = {1.0, Uy, y2 + ths, Uy * (y2 + t3), mad(y2, mad(6.0, ths, y2), tt)};
  const double dx[5] = {0.0, 1.0, 2.0 * Ux, 3.0 * hx[2], 4.0 * hx[3]};
  const double dy[5] = {0.0, 1.0, 2.0 * Uy, 3.0 * hy[2], 4.0 * hy[3]};
  const double tx[5] = {0.0, 0.0, 1.0, 3.0 * Ux, 6.0 * hx[2]};
  const double ty[5] = {0.0, 0.0, 1.0, 3.0 * Uy, 6.0 * hy[2]};
  double gr = 0.0, gx = 0.0, gy = 0.0, gt = 0.0;
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    // rows over q: sum_q L_pq h_q, sum_q L_pq dh_q/dU, sum_q L_pq dh_q/dTh
    double r = L[slot(p, 0)], ru = 0.0, rt = 0.0;
#pragma unroll
    for (int q = 1; p + q < 5; ++q) {
      const double l = L[slot(p, q)];
      r = mad(l, hy[q], r);
      ru = q == 1 ? l : mad(l, dy[q], ru);
      if (q == 2) rt = l;
      if (q > 2) rt = mad(l, ty[q], rt);
    }
    gr = p == 0 ? r : mad(hx[p], r, gr);
    if (p == 1) gx = r;
    if (p > 1) gx = mad(dx[p], r, gx);
    if (p < 4) gy = p == 0 ? ru : mad(hx[p], ru, gy);
    if (p < 3) gt = p == 0 ? rt : mad(hx[p], rt, gt);
    if (p > 1) gt = mad(tx[p], r, gt);
  }
  const double om = P.omega, orho = om * rho;
  gr *= om;
  gx *= orho;
  gy *= orho;
  gt *= orho;
  const double g00 = gr - (mad(ux, gx, uy * gy) - gt * mad(0.5, u2, -th)) * inv;
  const double g10 = mad(-ux, gt, gx) * inv;
  const double g01 = mad(-uy, gt, gy) * inv;
  const double ge2 = 0.5 * gt * inv;
  const double keep = 1.0 - om;
#pragma unroll
  for (int k = 0; k < NC; ++k) L[k] = keep * L[k];
  L[slot(0, 0)] += g00;
  L[slot(1, 0)] += g10;
  L[slot(0, 1)] += g01;
  L[slot(2, 0)] += ge2;
  L[slot(0, 2)] += ge2;
}

__device__ __forceinline__ void wall_adjoint(double (&B)[NC], const WallTable& wt, int i) {
  double su = 0.0;
#pragma unroll
  for (int k = 0; k < NC; ++k) su = mad(B[k], wt.v[i][k], su);
  B[slot(0, 0)] = mad(su, wt.ivk[i], B[slot(0, 0)]);
}

}  // namespace d2q37
