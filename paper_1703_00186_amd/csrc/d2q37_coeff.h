// Device code of the coefficient form of the lattice state.
//
// After a collision with the Hermite projection (Sec. 2) the 37 populations
// of a site are the weights times a polynomial of degree four in the hop:
//   f_l = w_l sum_ij c_ij e_lx^i e_ly^j,  i + j <= 4  (15 coefficients).
// The coefficient form stores those 15 FP64 numbers instead of the 37
// populations (120 instead of 296 bytes per site); a reader rebuilds a
// population from its source site's coefficients.  The arriving populations
// enter a regularized collision only through their 15 moments
//   m_ij = sum_l f_l e_lx^i e_ly^j,
// so those are what a reader sums up.  Powers of the integer hops cost far
// less than Hermite polynomials of the scaled velocities c_l = r e_l: most of
// the factors are 1, 2, 3, 4, 8, 9, .. (additions, or constants the
// instructions hold), where the Hermite values are 64-bit constants that do
// not fit the scalar registers all at once.
//
// The Hermite projection lives in to_poly, the step from moments to
// coefficients: with the moments of w itself (Gaussian up to degree eight),
// m = Gram c, so c = Gram^-1 m; to_poly goes through the scaled Hermite
// coefficients.  Gram is symmetric, and so the adjoint, which needs the
// transposed map, uses to_poly as well: its mu = B^T C^T lambda is
//   mu_l = sum_ij C_ij e_lx^i e_ly^j
// (times zero for the populations a wall supplied, which no reader asks for),
// stored the same way, and lambda enters through
//   M_ij = sum_l w_l lambda_l e_lx^i e_ly^j.
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

// Storage order of the exponents (i, j): the twelve that carry the
// macroscopic fields in the first six pair planes.
constexpr int kCI[NC] = {0, 2, 0, 4, 0, 2, 1, 3, 1, 0, 0, 2, 1, 3, 1};
constexpr int kCJ[NC] = {0, 0, 2, 0, 4, 2, 0, 0, 2, 1, 3, 1, 1, 1, 3};
__host__ __device__ constexpr int slot(int i, int j) {
  for (int k = 0; k < NC; ++k)
    if (kCI[k] == i && kCJ[k] == j) return k;
  return -1;
}
__host__ __device__ constexpr double ipow(int e, int n) {
  double v = 1.0;
  for (int k = 0; k < n; ++k) v *= e;
  return v;
}

// Geometry of a coefficient buffer: no halos.  Column x is cs doubles long:
// seven planes of pairs, [pitch rows][2] (16-byte accesses), then one plane
// of single values (slot 14).
struct CGeom {
  int lx, ly;
  int periodic;     // periodic y (rows wrap), else walls
  int nw;           // waves that cover a column
  int stream;       // columns are stored past the caches
  unsigned pitch;   // rows of a plane (ly rounded up to 32)
  long long cs;     // NC * pitch
};
__host__ __device__ __forceinline__ CGeom coeff_geom(const Geom& g) {
  CGeom c{};  // what the site kernels use
  c.lx = g.lx;
  c.ly = g.ly;
  c.periodic = !g.walls;
  c.pitch = unsigned((g.ly + 31) / 32 * 32);
  c.cs = (long long)NC * c.pitch;
  return c;
}

// A state buffer in this form starts with a header of 256 bytes: the word that
// names the form, and in the second and third double the wall temperatures of
// kFormCoeffWalls.
constexpr int kDataOffset = 32;  // doubles
__host__ __device__ __forceinline__ const double* coeffs(const void* buf) {
  return static_cast<const double*>(buf) + kDataOffset;
}
__host__ __device__ __forceinline__ double* coeffs(void* buf) {
  return static_cast<double*>(buf) + kDataOffset;
}

// Collision parameters in hop units (velocities over r, temperatures over r^2).
struct CPhys {
  double omega, keep;  // 1 / tau, 1 - 1 / tau
  double gx, gy;       // tau g / r
  double dt;           // temperature shift / r^2
};
inline CPhys make_cphys(const Phys& p) {
  return {p.omega, 1.0 - p.omega, p.tau_gx / R, p.tau_gy / R, p.dtheta / R2};
}

// The walls in moment space.  A wall row's unknown populations are rho_w v_l
// (Sec. 2: fixed temperature, zero velocity), so they add rho_w V_ij,
// V_ij = sum over the unknown l of v_l e_lx^i e_ly^j, to the moments of the
// known ones; rho_w = m_00(known) / sum over the known l of v_l.  Rows 0..2
// from the bottom, then ly - 3 .. ly - 1.
struct WallTable {
  double v[6][NC];  // V_ij in storage order
  double ivk[6];    // 1 / sum over the known l of v_l
};

// V_ij and sum_known v are quadratic in th = T_wall - 1: their coefficients.
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
          b.v[n][i][k] += v[n] * ipow(EX[l], kCI[k]) * ipow(EY[l], kCJ[k]);
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

// The two uses of the expansion and its transpose: where the weights go.
struct Forward {
  static __host__ __device__ constexpr double wup(int l) { return W[l]; }
  static __host__ __device__ constexpr double wdown(int) { return 1.0; }
};
struct Adjoint {
  static __host__ __device__ constexpr double wup(int) { return 1.0; }
  static __host__ __device__ constexpr double wdown(int l) { return W[l]; }
};

// y + c x for the constant factors of the sums
template <class T>
__device__ __forceinline__ double add_scaled(T c, double x, double y) {
  return c == 1.0 ? y + x : c == -1.0 ? y - x : mad(c, x, y);
}

// P_j = sum_i c_ij ex^i
template <int ex>
__device__ __forceinline__ void column_sums(const double (&c)[NC], double (&P)[5]) {
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    double s = c[slot(0, j)];
#pragma unroll
    for (int i = 1; i + j < 5; ++i)
      if (ex != 0) s = add_scaled(ipow(ex, i), c[slot(i, j)], s);
    P[j] = s;
  }
}

// populations (ex, 0) and (ex, +-k) from the column sums: the parts even and
// odd in e_y once, then their sum and difference
template <class K, int ex>
__device__ __forceinline__ double population0(const double (&P)[5]) {
  constexpr double w = K::wup(label(ex, 0));
  return w == 1.0 ? P[0] : w * P[0];
}
template <class K, int ex, int k>
__device__ __forceinline__ void populations(const double (&P)[5], double& plus, double& minus) {
  constexpr double w = K::wup(label(ex, k)), wk = w * k;
  double e = add_scaled(ipow(k, 4), P[4], add_scaled(ipow(k, 2), P[2], P[0]));
  const double o = add_scaled(ipow(k, 2), P[3], P[1]);
  if (w != 1.0) e = w * e;
  plus = add_scaled(wk, o, e);
  minus = add_scaled(-wk, o, e);
}

// One e_x group of a site's arriving populations: (ex, 0) and (ex, +-k).
struct Group {
  double zero, plus[3], minus[3];
};

// s_j += contributions of (ex, +-k)
template <class K, int ex, int k>
__device__ __forceinline__ void project_pairs(const Group& f, double (&s)[5]) {
  constexpr double w = K::wdown(label(ex, k));
  double sum = f.plus[k - 1] + f.minus[k - 1], dif = f.plus[k - 1] - f.minus[k - 1];
  if (w != 1.0) {
    sum = w * sum;
    dif = w * dif;
  }
  s[0] = s[0] + sum;
  s[1] = k == 1 ? dif : mad(ipow(k, 1), dif, s[1]);
  s[2] = k == 1 ? sum : mad(ipow(k, 2), sum, s[2]);
  s[3] = k == 1 ? dif : mad(ipow(k, 3), dif, s[3]);
  s[4] = k == 1 ? sum : mad(ipow(k, 4), sum, s[4]);
  if constexpr (k < reach(ex)) project_pairs<K, ex, k + 1>(f, s);
}

// m_ij += contribution of the group; groups arrive with ex = 3 first (which
// starts the sums), then 2, ... -3
template <class K, int ex>
__device__ __forceinline__ void project_group(const Group& f, double (&m)[NC]) {
  constexpr double w = K::wdown(label(ex, 0));
  double s[5] = {w == 1.0 ? f.zero : w * f.zero, 0.0, 0.0, 0.0, 0.0};
  project_pairs<K, ex, 1>(f, s);
#pragma unroll
  for (int i = 0; i < (ex == 0 ? 1 : 5); ++i) {
    const double h = ipow(ex, i);
#pragma unroll
    for (int j = 0; i + j < 5; ++j) {
      double& t = m[slot(i, j)];
      if (ex == 3)
        t = i == 0 ? s[j] : h * s[j];
      else
        t = add_scaled(h, s[j], t);
    }
  }
}

// the populations of one e_x group of a site from its coefficients
template <class K, int ex>
__device__ __forceinline__ void expand_group(const double (&c)[NC], Group& f) {
  double P[5];
  column_sums<ex>(c, P);
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

// all 37 populations of a site <-> its coefficients / their moments
template <class K, int ex = 3>
__device__ __forceinline__ void expand_site(const double (&c)[NC], double (&v)[Q]) {
  Group f;
  expand_group<K, ex>(c, f);
  to_labels<ex>(f, v);
  if constexpr (ex > -3) expand_site<K, ex - 1>(c, v);
}
template <class K, int ex = 3>
__device__ __forceinline__ void project_site(const double (&v)[Q], double (&m)[NC]) {
  Group f;
  from_labels<ex>(v, f);
  project_group<K, ex>(f, m);
  if constexpr (ex > -3) project_site<K, ex - 1>(v, m);
}

// One site of a buffer (the readers' access; a wave's is in d2q37_coeff.hip).
typedef double v2d __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void load_coeffs(const double* __restrict__ src, const CGeom& g, int x,
                                            int y, double (&b)[NC]) {
  const double* col = src + x * g.cs;
#pragma unroll
  for (int m = 0; m < NC / 2; ++m) {
    const v2d d = *reinterpret_cast<const v2d*>(col + 2 * m * (long long)g.pitch + 2 * y);
    b[2 * m] = d.x;
    b[2 * m + 1] = d.y;
  }
  b[NC - 1] = col[(NC - 1) * (long long)g.pitch + y];
}

// fn(l, f_l) for the 37 populations of a site, one e_x group after the other
template <class Fn, int ex = 3>
__device__ __forceinline__ void each_population(const double (&c)[NC], const Fn& fn) {
  Group f;
  expand_group<Forward, ex>(c, f);
  fn(label(ex, 0), f.zero);
#pragma unroll
  for (int k = 1; k <= reach(ex); ++k) {
    fn(label(ex, -k), f.minus[k - 1]);
    fn(label(ex, k), f.plus[k - 1]);
  }
  if constexpr (ex > -3) each_population<Fn, ex - 1>(c, fn);
}

// A site that bc was applied to after its coefficients were stored (a scratch
// buffer, word form): the temperature of its wall.
__device__ __forceinline__ bool walls_since(const void* buf, unsigned form, const Geom& g, int y,
                                            double& th) {
  if (form != unsigned(kFormCoeffWalls)) return false;
  th = static_cast<const double*>(buf)[y < 3 ? 1 : 2];
  return y < 3 || y >= g.ly - 3;
}

// The 37 populations of a site of a scratch buffer that holds coefficients.
__device__ __forceinline__ void scratch_site(const void* buf, const Geom& g, int x, int y,
                                             double (&v)[Q]) {
  double c[NC], th;
  load_coeffs(coeffs(buf), coeff_geom(g), x, y, c);
  expand_site<Forward>(c, v);
  if (walls_since(buf, *static_cast<const unsigned*>(buf), g, y, th))
    wall_site<double>(v, y, g.ly, th, th, 0.0);
}

// Population l of a site.
template <int l>
__device__ __forceinline__ double population(const double (&c)[NC]) {
  constexpr int ex = EX[l], ey = EY[l];
  double P[5], plus, minus;
  column_sums<ex>(c, P);
  if constexpr (ey == 0) return population0<Forward, ex>(P);
  populations<Forward, ex, (ey < 0 ? -ey : ey)>(P, plus, minus);
  return ey > 0 ? plus : minus;
}

// propagate from coefficients: fn(l, f_l) for the populations that arrive at a
// site, each from all 15 coefficients of the site it comes from (0 for those
// that a wall will supply).  4.4 KB of loads a site, from the caches: as slow as
// a few steps, for the first step after the collision changed.  One population
// after the other, which leaves the registers of the kernels it stands in alone.
template <int l = 0, class Fn>
__device__ __forceinline__ void gather_coeffs(const double* src, const CGeom& g, int x, int y,
                                              const Fn& fn) {
  int xs = x - EX[l], ys = y - EY[l];
  xs = xs < 0 ? xs + g.lx : (xs >= g.lx ? xs - g.lx : xs);
  const bool outside = ys < 0 || ys >= g.ly;
  if (outside) ys = !g.periodic ? y : ys < 0 ? ys + g.ly : ys - g.ly;
  double c[NC];
  load_coeffs(src, g, xs, ys, c);
  double v = population<l>(c);
  asm volatile("" : "+s"(src), "+v"(v));  // the next site's loads stay behind this
  fn(l, outside && !g.periodic ? 0.0 : v);
  if constexpr (l + 1 < Q) gather_coeffs<l + 1>(src, g, x, y, fn);
}

// Hermite coefficients scaled by r^(p+q) / (p! q!) -> polynomial coefficients,
// in place (the leading ones are the same; lower ones get the tails of He_n),
// the second ones from s b_20 and s b_02.
// c_00 comes last, as what the others leave of the mass with the weights'
// moments G20 = sum w e_x^2 (about r^-2), G40 = sum w e_x^4 (3 r^-4) and
// G22 = sum w e_x^2 e_y^2 (r^-4): their rounding then does not touch it.
__device__ __forceinline__ void add_tails(double (&b)[NC], double s = 1.0) {
  const double c40 = b[slot(4, 0)], c04 = b[slot(0, 4)], c22 = b[slot(2, 2)];
  const double tail = -IR2 * c22;
  const double c20 = mad(s, b[slot(2, 0)], mad(-IR2_6, c40, tail));
  const double c02 = mad(s, b[slot(0, 2)], mad(-IR2_6, c04, tail));
  b[slot(2, 0)] = c20;
  b[slot(0, 2)] = c02;
  b[slot(0, 0)] = b[slot(0, 0)] - mad(G20, c20 + c02, mad(G40, c40 + c04, G22 * c22));
  b[slot(1, 1)] = mad(-IR2_3, b[slot(3, 1)] + b[slot(1, 3)], b[slot(1, 1)]);
  b[slot(1, 0)] = mad(-IR2_3, b[slot(3, 0)], mad(-IR2, b[slot(1, 2)], b[slot(1, 0)]));
  b[slot(0, 1)] = mad(-IR2_3, b[slot(0, 3)], mad(-IR2, b[slot(2, 1)], b[slot(0, 1)]));
}

// c = Gram^-1 m: moments -> coefficients of the polynomial with those moments,
// the second ones centred: m_20 - G20 m_00 (zero at rest with T = 1).
//
// What is conserved has to come back as it went in, or a run gains a little of
// it at every step: a relative error of 1e-16 a step in the energy is more than
// all of the run's rounding after some ten.  So the constants are rounded once
// (powers of r built up from a rounded r cost 4e-16 of the energy at T = 1.5), and
// the energy is relaxed and mapped as its distance from that of T = 1, which
// leaves 6e-17 of the constants' rounding at T = 0.5 and 1e-17 at 1.  Against an
// extended-precision run, 256 x 128 after 50 steps: T 1.2e-14 to 1.9e-15 (rms),
// rho 9.2e-15 to 2.7e-15, u 4.1e-13 to 8.7e-14 of the largest; gradients of
// the kinetic energy after 20 to 40 steps 4.7e-14 to 1.2e-14.  1920 x 2048: 3463 and
// 3477 us for 20 steps with their start and results.
__device__ __forceinline__ double centred(double m20, double m00) { return mad(-G20, m00, m20); }
__device__ __forceinline__ void to_poly_centred(double (&m)[NC]) {
  const double m00 = m[slot(0, 0)], m10 = m[slot(1, 0)], m01 = m[slot(0, 1)];
  const double t20 = m[slot(2, 0)], t02 = m[slot(0, 2)], m11 = m[slot(1, 1)];
  // r^4/24 (r^4 m40 - 6 r^2 m20 + 3 m00), ...
  m[slot(4, 0)] = mad(R8_24, m[slot(4, 0)], mad(-R6 / 4.0, t20, (-R4 / 8.0) * m00));
  m[slot(0, 4)] = mad(R8_24, m[slot(0, 4)], mad(-R6 / 4.0, t02, (-R4 / 8.0) * m00));
  m[slot(2, 2)] = mad(R8 / 4.0, m[slot(2, 2)], mad(-R6 / 4.0, t20 + t02, (-R4 / 4.0) * m00));
  m[slot(3, 1)] = mad(R8_6, m[slot(3, 1)], (-R6 / 2.0) * m11);
  m[slot(1, 3)] = mad(R8_6, m[slot(1, 3)], (-R6 / 2.0) * m11);
  // r^3/6 (r^3 m30 - 3 r m10), r^3/2 (r^3 m21 - r m01), ...
  m[slot(3, 0)] = mad(R6_6, m[slot(3, 0)], (-R4 / 2.0) * m10);
  m[slot(0, 3)] = mad(R6_6, m[slot(0, 3)], (-R4 / 2.0) * m01);
  m[slot(2, 1)] = mad(R6 / 2.0, m[slot(2, 1)], (-R4 / 2.0) * m01);
  m[slot(1, 2)] = mad(R6 / 2.0, m[slot(1, 2)], (-R4 / 2.0) * m10);
  // r^4 m11, r^2 m10; the second ones are r^4/2 t20, r^4/2 t02
  m[slot(1, 1)] = R4 * m11;
  m[slot(1, 0)] = R2 * m10;
  m[slot(0, 1)] = R2 * m01;
  add_tails(m, R4 / 2.0);
}
__device__ __forceinline__ void to_poly(double (&m)[NC]) {
  m[slot(2, 0)] = centred(m[slot(2, 0)], m[slot(0, 0)]);
  m[slot(0, 2)] = centred(m[slot(0, 2)], m[slot(0, 0)]);
  to_poly_centred(m);
}

// The walls: m holds the moments of the known populations.
__device__ __forceinline__ void wall_moments(double (&m)[NC], const WallTable& wt, int i) {
  const double rho_w = m[0] * wt.ivk[i];
#pragma unroll
  for (int k = 0; k < NC; ++k) m[k] = mad(rho_w, wt.v[i][k], m[k]);
}

// collide: the moments m_ij of the arriving populations become the
// coefficients c_ij of the collided ones.  Eq. (2) moments; the equilibrium
// has the raw moments rho G_i(U_x) G_j(U_y) of a Gaussian up to order four
// (G_0..4 = 1, U, U^2 + T, U^3 + 3 U T, U^4 + 6 U^2 T + 3 T^2), taken at the
// forced U and T; relaxation with rate omega, then the projection.  Mass is
// conserved exactly (m_00 is not touched); m_20 and m_02 are relaxed centred.
__device__ __forceinline__ void collide_moments(double (&m)[NC], const CPhys& P) {
  const double rho = m[slot(0, 0)], inv = 1.0 / rho;
  const double ux = m[slot(1, 0)] * inv, uy = m[slot(0, 1)] * inv;
  m[slot(2, 0)] = centred(m[slot(2, 0)], rho);
  m[slot(0, 2)] = centred(m[slot(0, 2)], rho);
  // T - G20, before and after the forcing
  const double d0 = 0.5 * mad(m[slot(2, 0)] + m[slot(0, 2)], inv, -mad(ux, ux, uy * uy));
  const double Ux = ux + P.gx, Uy = uy + P.gy, d = d0 + P.dt, T = d + G20;
  const double x2 = Ux * Ux, y2 = Uy * Uy, t3 = 3.0 * T, tt = t3 * T;
  const double gx[5] = {1.0, Ux, x2 + T, Ux * (x2 + t3), mad(x2, mad(6.0, T, x2), tt)};
  const double gy[5] = {1.0, Uy, y2 + T, Uy * (y2 + t3), mad(y2, mad(6.0, T, y2), tt)};
  const double om_rho = P.omega * rho;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const double r = i == 0 ? om_rho : om_rho * gx[i];
#pragma unroll
    for (int j = 0; i + j < 5; ++j) {
      if (i + j == 0) continue;
      double& t = m[slot(i, j)];
      if (i == 2 && j == 0)
        t = mad(om_rho, x2 + d, P.keep * t);
      else if (i == 0 && j == 2)
        t = mad(om_rho, y2 + d, P.keep * t);
      else
        t = j == 0 ? mad(P.keep, t, r) : mad(r, gy[j], P.keep * t);
    }
  }
  to_poly_centred(m);
}

// Eq. (2) fields of a site from its coefficients (the first twelve).
__device__ __forceinline__ Macro macro_coeffs(const double (&c)[12]) {
  const double c00 = c[slot(0, 0)], c2s = c[slot(2, 0)] + c[slot(0, 2)];
  const double c4s = c[slot(4, 0)] + c[slot(0, 4)], c22 = c[slot(2, 2)];
  const double m10 = mad(G22, c[slot(1, 2)], mad(G40, c[slot(3, 0)], G20 * c[slot(1, 0)]));
  const double m01 = mad(G22, c[slot(2, 1)], mad(G40, c[slot(0, 3)], G20 * c[slot(0, 1)]));
  Macro f;
  f.rho = mad(G22, c22, mad(G40, c4s, mad(G20, c2s, c00)));
  // (sum |c|^2 f) / 2 - rho, zero at rest with T = 1
  const double e = mad(2.0 * G22, c22, mad(2.0 * G40, c4s, IR2 * c2s));
  f.inv_rho = 1.0 / f.rho;
  f.ux = R * m10 * f.inv_rho;
  f.uy = R * m01 * f.inv_rho;
  f.th = mad(e, f.inv_rho, -0.5 * mad(f.ux, f.ux, f.uy * f.uy));
  return f;
}

// B^T C^T of a site: M holds sum_l w_l lambda_l e^ij at the site's arriving
// populations, (rho, jx, jy, e) the pre-collision moments of the tape (rho,
// rho u, sum |c|^2 f); on return M holds the coefficients C_ij of mu.
__device__ __forceinline__ void adjoint_moments(double (&M)[NC], double rho, double jx, double jy,
                                                double e, const CPhys& P) {
  to_poly(M);  // now the gradient with respect to the relaxed moments
  const double inv = 1.0 / rho;
  const double ux = (jx * (1.0 / R)) * inv, uy = (jy * (1.0 / R)) * inv;
  const double u2 = mad(ux, ux, uy * uy);
  const double t0 = 0.5 * mad(e * IR2, inv, -u2);
  const double Ux = ux + P.gx, Uy = uy + P.gy, T = t0 + P.dt;
  // G_n, dG_n/dU = n G_(n-1), dG_n/dT = n (n - 1) / 2 G_(n-2) of both directions
  const double x2 = Ux * Ux, y2 = Uy * Uy, t3 = 3.0 * T, tt = t3 * T;
  const double hx[5] = {1.0, Ux, x2 + T, Ux * (x2 + t3), mad(x2, mad(6.0, T, x2), tt)};
  const double hy[5] = {1.0, Uy, y2 + T, Uy * (y2 + t3), mad(y2, mad(6.0, T, y2), tt)};
  const double dx[5] = {0.0, 1.0, 2.0 * Ux, 3.0 * hx[2], 4.0 * hx[3]};
  const double dy[5] = {0.0, 1.0, 2.0 * Uy, 3.0 * hy[2], 4.0 * hy[3]};
  const double tx[5] = {0.0, 0.0, 1.0, 3.0 * Ux, 6.0 * hx[2]};
  const double ty[5] = {0.0, 0.0, 1.0, 3.0 * Uy, 6.0 * hy[2]};
  double gr = 0.0, gx = 0.0, gy = 0.0, gt = 0.0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    // over j: sum M_ij G_j, sum M_ij dG_j/dU, sum M_ij dG_j/dT
    double r = M[slot(i, 0)], ru = 0.0, rt = 0.0;
#pragma unroll
    for (int j = 1; i + j < 5; ++j) {
      const double l = M[slot(i, j)];
      r = mad(l, hy[j], r);
      ru = j == 1 ? l : mad(l, dy[j], ru);
      if (j == 2) rt = l;
      if (j > 2) rt = mad(l, ty[j], rt);
    }
    gr = i == 0 ? r : mad(hx[i], r, gr);
    if (i == 1) gx = r;
    if (i > 1) gx = mad(dx[i], r, gx);
    if (i < 4) gy = i == 0 ? ru : mad(hx[i], ru, gy);
    if (i < 3) gt = i == 0 ? rt : mad(hx[i], rt, gt);
    if (i > 1) gt = mad(tx[i], r, gt);
  }
  const double om_rho = P.omega * rho;
  gr *= P.omega;
  gx *= om_rho;
  gy *= om_rho;
  gt *= om_rho;
#pragma unroll
  for (int k = 0; k < NC; ++k) M[k] = P.keep * M[k];
  M[slot(0, 0)] += gr - (mad(ux, gx, uy * gy) - gt * mad(0.5, u2, -t0)) * inv;
  M[slot(1, 0)] += mad(-ux, gt, gx) * inv;
  M[slot(0, 1)] += mad(-uy, gt, gy) * inv;
  const double ge = 0.5 * gt * inv;
  M[slot(2, 0)] += ge;
  M[slot(0, 2)] += ge;
}

// the share of the unknown populations' adjoint (their sum weighted by v_l,
// over sum_known v) that every known one gets: a shift of C_00
__device__ __forceinline__ void wall_adjoint(double (&C)[NC], const WallTable& wt, int i) {
  double su = 0.0;
#pragma unroll
  for (int k = 0; k < NC; ++k) su = mad(C[k], wt.v[i][k], su);
  C[slot(0, 0)] = mad(su, wt.ivk[i], C[slot(0, 0)]);
}

// The readers' share of a site (twelve coefficients, 96 bytes).
__device__ __forceinline__ Macro load_macro(const double* __restrict__ src, const CGeom& g, int x,
                                            int y) {
  const double* col = src + x * g.cs + 2 * y;
  double c[12];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const v2d d = *reinterpret_cast<const v2d*>(col + 2 * m * (long long)g.pitch);
    c[2 * m] = d.x;
    c[2 * m + 1] = d.y;
  }
  return macro_coeffs(c);
}

// As k_obs_rows: the sums over the columns x0 .. x1 - 1 of a row.
__device__ __forceinline__ void sum_observables(const double* __restrict__ src, const CGeom& g,
                                                int y, int x0, int x1, double (&acc)[6]) {
#pragma unroll 4
  for (int x = x0; x < x1; ++x) {
    const Macro m = load_macro(src, g, x, y);
    const double T = 1.0 + m.th;
    acc[0] += m.rho;
    acc[1] += m.ux;
    acc[2] += m.uy;
    acc[3] += T;
    acc[4] += 0.5 * m.rho * (m.ux * m.ux + m.uy * m.uy);
    acc[5] += m.rho * T;
  }
}

// A site's kinetic energy, and its derivative with respect to population l.
__device__ __forceinline__ double kinetic(const Macro& m) {
  return 0.5 * m.rho * (m.ux * m.ux + m.uy * m.uy);
}
__device__ __forceinline__ double kinetic_slope(const Macro& m, int l) {
  return R * (EX[l] * m.ux + EY[l] * m.uy) - 0.5 * (m.ux * m.ux + m.uy * m.uy);
}

}  // namespace d2q37

#pragma clang fp contract(fast)  // as the rest of the code is compiled
