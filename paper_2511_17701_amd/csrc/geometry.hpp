// geometry.hpp -- grid description and Kerr-Schild 3+1 geometry in code
// coordinates, evaluated on the device (and on the host for dt and tables).
//
// Code coordinates (App. A, quasi-spherical Kerr-Schild): r = r0 + exp(xi),
//   xi = xi_min + x1 dxi; theta = eta + 2 h0 eta (pi - 2 eta)(pi - eta) / pi^2,
//   eta = x2 dth (dth is the uniform eta spacing); phi with dphi = 1.
//   r0 = h0 = 0 is the logarithmic-r, uniform-theta grid.
// Kerr-Schild 3+1 split (Sec. 2.1, App. A), with S2 = Sigma + 2 M r:
//   Sigma = r^2 + a^2 cos^2, Delta = r^2 - 2 M r + a^2,
//   A = (r^2 + a^2)^2 - a^2 Delta sin^2, alpha^2 = Sigma / S2,
//   beta^r = 2 M r / S2, h^rr = A / (Sigma S2), h^rphi = a / Sigma,
//   h^thth = 1 / Sigma, h^phiphi = 1 / (Sigma sin^2),
//   h_rr = S2 / Sigma, h_rphi = -a (S2 / Sigma) sin^2, h_thth = Sigma,
//   h_phiphi = A sin^2 / Sigma, sqrt(h) = Sigma sin / alpha.
// A covariant index 1 carries a factor R = dr/dx1 = dxi (r - r0), index 2 a
// factor T = dtheta/dx2; contravariant indices the inverse factors.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace grpic {

constexpr double kPi = 3.14159265358979323846;

// Uniform values of the particle update in its own precision.  The single-
// precision copy is made on the host: a conversion of a kernel argument is a
// vector instruction at a quarter of the full rate in every wavefront.
template <class R>
struct UniT {
  R a, a2, M, two_M;
  R dxi, dth, inv_dth2;
  R dt, inv_dt, charge_scale, small_angle;
};

// Everything a kernel needs to know about the grid and the run, by value.
struct Grid {
  double a, M;
  double xi_min, dxi, dth, inv_dth, inv_dth2;  // xi_min = log(r_min - r0); dth: eta spacing
  double r0, h0;                      // quasi-spherical map (0, 0: log r, uniform theta)
  double dt, inv_dt;
  double small_angle;
  double charge_scale;
  double iter_tol;  // relative FP64 convergence test of the implicit iterations (0: off)
  // sin, cos of the clamped polar angles small_angle and pi - small_angle
  double sin_lo, cos_lo, sin_hi, cos_hi;
  int n_r, n_th, ng, ld;  // ld = n_th + 2 ng (row length of a plane)
  int n_iter, n_filter, n_absorb;
  int ser;                // series used by the push for in-cell offsets (0 = library)
  double axis_band;       // short series: polar band next to each axis (4 cells)
  // uniform values the push would otherwise form per wavefront in vector
  // registers: a^2, 2 M, pi - small_angle, pi - axis_band
  double a2, two_M, th_hi, band_hi;
  int i_fp64;             // single-precision push: cells i1 < i_fp64 (r < 3 M, the
                          // horizon region) take the metric and its derivatives in FP64
  // cells at least this far from both axes take the push's table form of the
  // polar angle in double / single precision (outside the series' axis bands)
  int mid64, mid32;
  // the gather's 32-bit byte offsets and 24-bit index product hold (planes
  // below 4 GiB, rows and columns below 2^24)
  int narrow;
  UniT<float> uf;
  int64_t plane;          // reals per plane
};

__host__ __device__ inline int64_t ix(const Grid& g, int i, int j) {
  return (int64_t)(i + g.ng) * g.ld + (j + g.ng);
}

// 1-D coordinate tables, indexed by (index + ng); [0] integer, [1] half-integer
// points: r and 1/(R deta) along x1 (R = dr/dx1, deta the eta spacing); sin,
// cos, 1/sin (0 on the axis), T = dtheta/dx2 and deta/T along x2 (T = deta and
// deta/T = 1 when h0 = 0).  rf: r - r0 at integer x1, sf, cf: sin, cos at
// integer x2, in single precision.
struct Tables {
  const double* __restrict__ r[2];
  const double* __restrict__ ird[2];
  const double* __restrict__ s[2];
  const double* __restrict__ c[2];
  const double* __restrict__ is[2];
  const double* __restrict__ td[2];
  const double* __restrict__ eta_t[2];
  const float* __restrict__ rf;
  const float* __restrict__ sf;
  const float* __restrict__ cf;
};

// The type of the constants that go with a value type (tangent.hpp: its
// numbers take plain constants).
template <class R>
struct ScalarOf {
  using type = R;
};
template <class R>
using Scalar = typename ScalarOf<R>::type;

template <class R>
__host__ __device__ inline UniT<Scalar<R>> uni(const Grid& g) {
  if constexpr (sizeof(Scalar<R>) == 4) return g.uf;
  else return {g.a, g.a2, g.M, g.two_M, g.dxi, g.dth, g.inv_dth2, g.dt, g.inv_dt, g.charge_scale, g.small_angle};
}

// Element k of a table or array by a 32-bit byte offset from a uniform base
// (k sizeof(T) below 2^32): one address register, no 64-bit vector arithmetic.
template <class T>
__device__ inline T& elem(T* __restrict__ p, uint32_t k) {
  return *(T*)((char*)p + (size_t)(uint32_t)(k * (uint32_t)sizeof(T)));
}

// Pusher coefficients at a point: lapse, shift and inverse spatial metric.
template <class R>
struct CoeffsT {
  R alpha, beta1, hu11, hu22, hu33, hu13;
};

// Coefficients plus the tetrad factors of App. A at a point, as the EM stage
// uses them: is11 = 1/sqrt(h^11), s22 = sqrt(h_22), s33 = sqrt(h_33) and its
// inverse.  The others follow: sqrt(h^11) = h^11 is11, 1/sqrt(h_22) = h^22 s22
// and h_13 / h_33 = -h^13 is11^2, so the stage divides by nothing.
template <class R>
struct FrameT {
  CoeffsT<R> c;
  R is11, s22, s33, is33;
};

// First derivatives of the pusher coefficients: d/dx1 ([0]) and d/dx2 ([1]) of
// the lapse and the shift; of the inverse metric the logarithmic ones, which
// the force takes as factors of its own terms h^jk u_j u_k:
//   d ln h^11 = l11,  d ln h^22 = -z - (0, tt),  d ln h^33 = -z - (0, ct),
//   d ln h^13 = -z - (dxi, 0),
// z = d ln Sigma, ct = 2 T cot(theta), tt = 2 d ln T / dx2.
template <class R>
struct GradT {
  R alpha[2], beta1[2], l11[2], z[2], ct, tt;
};

// r, sin(theta), cos(theta) of a point, and the map factors there:
// rd = dr/dx1, td = dtheta/dx2, itd2 = 1/td^2, dtd = d td / dx2
template <class R>
struct RSCT {
  R r, s, c;
  R rd, td, itd2, dtd;
};

using Coeffs = CoeffsT<double>;
using Frame = FrameT<double>;
using Grad = GradT<double>;
using RSC = RSCT<double>;

__host__ __device__ inline double clamp_theta(const Grid& g, double th) {
  return fmin(fmax(th, g.small_angle), kPi - g.small_angle);
}

__host__ __device__ inline void sin_cos(double th, double* s, double* c) {
#ifdef __HIP_DEVICE_COMPILE__
  sincos(th, s, c);
#else
  *s = std::sin(th);
  *c = std::cos(th);
#endif
}

// a b + k with a literal k.  A 64-bit literal has no encoding in a vector
// instruction: the compiler puts it in a vector register pair (two moves) for
// each use; as a scalar operand it costs the vector unit nothing.
__device__ inline double fma_k(double a, double b, double k) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
  return r;
}

// 1/x and 1/sqrt(x) for positive normal x: hardware seeds (relative error
// below 2^-23 in double) refined on the device by one step of third order in
// double (error e^3 ~ 2^-69 before rounding; two Newton steps would take one
// and two operations more), by one Newton step in single (error ~1 ulp in
// both); plain division on the host.
__host__ __device__ inline double rcp(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
#else
  return 1.0 / x;
#endif
}

__host__ __device__ inline double rsqrt(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  // y (1 + e/2 + 3 e^2/8)
  return fma(y * e, fma(e, 0.375, 0.5), y);
#else
  return 1.0 / std::sqrt(x);
#endif
}

__host__ __device__ inline float rcp(float x) {
#ifdef __HIP_DEVICE_COMPILE__
  const float y = __builtin_amdgcn_rcpf(x);
  return fmaf(y, fmaf(-x, y, 1.0f), y);
#else
  return 1.0f / x;
#endif
}

__host__ __device__ inline float rsqrt(float x) {
#ifdef __HIP_DEVICE_COMPILE__
  const float y = __builtin_amdgcn_rsqf(x);
  return fmaf(y, fmaf(-0.5f * x * y, y, 0.5f), y);
#else
  return 1.0f / std::sqrt(x);
#endif
}

// The quasi-spherical map (App. A): r and R = dr/dx1 at x1; theta,
// T = dtheta/dx2 and dT/dx2 at x2.  Beyond either axis the polar map is
// continued by reflection (theta(-x2) = -theta(x2), theta(2 n_th - x2) =
// 2 pi - theta(x2)), so that geometry there mirrors the interior.
__host__ __device__ inline void map_r(const Grid& g, double x1, double* r, double* rd) {
  const double e = exp(g.xi_min + x1 * g.dxi);
  *r = g.r0 + e;
  *rd = g.dxi * e;
}

__host__ __device__ inline void map_theta(const Grid& g, double x2, double* th, double* td,
                                          double* dtd) {
#pragma clang fp contract(off)
  double sg = 1.0, off = 0.0;
  if (x2 < 0.0) {
    x2 = -x2;
    sg = -1.0;
  } else if (x2 > (double)g.n_th) {
    x2 = 2.0 * g.n_th - x2;
    sg = -1.0;
    off = 2.0 * kPi;
  }
  // theta is rounded from exactly these operations in this order (no fused
  // multiply-adds, a true division by pi^2): next to theta = pi one unit in
  // its last place is a relative 1e-13 of sin(theta) a few 1e-4 rad from the
  // axis, so every evaluation of the map must round alike
  const double eta = x2 * g.dth, y = eta * (1.0 / kPi), h0 = g.h0;
  *th = off + sg * (eta + 2.0 * h0 * eta * (kPi - 2.0 * eta) * (kPi - eta) / (kPi * kPi));
  *td = g.dth * (1.0 + 2.0 * h0 + 12.0 * h0 * y * (y - 1.0));
  *dtd = sg * g.dth * g.dth * 12.0 * h0 * (2.0 * y - 1.0) * (1.0 / kPi);
}

// r, clamped sin/cos and the map factors by the library functions
__host__ __device__ inline RSC rsc_direct(const Grid& g, double x1, double x2) {
  RSC p;
  map_r(g, x1, &p.r, &p.rd);
  double th;
  map_theta(g, x2, &th, &p.td, &p.dtd);
  const double it = rcp(p.td);
  p.itd2 = it * it;
  sin_cos(clamp_theta(g, th), &p.s, &p.c);
  return p;
}

// Inverse metric, lapse and shift at a point (R = dr/dx1).
__host__ __device__ inline Coeffs coeffs_from(const Grid& g, RSC p) {
  const double r = p.r, s = p.s, c = p.c;
  const double a = g.a, a2 = g.a2, r2 = r * r;
  const double tMr = g.two_M * r;
  const double Sig = r2 + a2 * c * c;
  const double S2 = Sig + tMr;
  const double ra = r2 + a2;
  const double s2 = s * s;
  const double A = ra * ra - a2 * (ra - tMr) * s2;
  const double Rr = p.rd;
  // one reciprocal for 1/Sigma, 1/S2, 1/sin^2 and 1/R
  const double q = rcp(Sig * S2 * s2 * Rr);
  const double iSig = S2 * s2 * Rr * q, iS2 = Sig * s2 * Rr * q;
  const double is2 = Sig * S2 * Rr * q, iR = Sig * S2 * s2 * q;
  Coeffs m;
  const double y = Sig * iS2;
  m.alpha = y * rsqrt(y);
  m.beta1 = tMr * iS2 * iR;
  m.hu11 = A * iSig * iS2 * iR * iR;
  m.hu13 = a * iSig * iR;
  m.hu22 = iSig * p.itd2;
  m.hu33 = iSig * is2;
  return m;
}

__host__ __device__ inline Coeffs coeffs_at(const Grid& g, double x1, double x2) {
  return coeffs_from(g, rsc_direct(g, x1, x2));
}

// Coefficients, tetrad factors and first derivatives at a point.  Three
// inverse square roots (of Sigma, S2 and A) and one reciprocal give them all.
// kMap: the general map (tt is 0 on the logarithmic-r, uniform-theta grid).
template <bool kMap, class R>
__host__ __device__ inline void frame_from(const Grid& g, RSCT<R> p, FrameT<R>* f, GradT<R>* d) {
  const R r = p.r, s = p.s, c = p.c, T = p.td, Rr = p.rd;
  using S = Scalar<R>;
  const UniT<S> U = uni<R>(g);
  const S a = U.a, M = U.M, dxi = U.dxi, a2 = U.a2;
  const R r2 = r * r;
  const R tMr = U.two_M * r;
  const R Sig = r2 + a2 * c * c;
  const R S2 = Sig + tMr;
  const R ra = r2 + a2;
  const R Del = ra - tMr;
  const R s2 = s * s;
  const R A = ra * ra - a2 * Del * s2;
  const R g1 = rsqrt(Sig), g2 = rsqrt(S2), gA = rsqrt(A);
  const R q = rcp(s2 * Rr);
  const R iR = s2 * q, is2 = Rr * q;
  const R iSig = g1 * g1, iS2 = g2 * g2, iA = gA * gA;
  const R rS = Sig * g1, rS2 = S2 * g2, rA = A * gA;  // square roots of Sigma, S2, A

  f->c.alpha = rS * g2;
  f->c.beta1 = tMr * iS2 * iR;
  const R hr = A * iSig * iS2 * iR;
  f->c.hu11 = hr * iR;
  f->c.hu13 = a * iSig * iR;
  f->c.hu22 = iSig * p.itd2;
  f->c.hu33 = iSig * is2;
  f->is11 = Rr * rS * rS2 * gA;
  f->s22 = rS * T;
  f->s33 = rA * g1 * s;
  f->is33 = rS * gA * s * is2;

  // radial and polar derivatives of Sigma and A (S2 shares dSigma/dtheta)
  const R dSig_t = (S)-2 * a2 * s * c;
  const R dA_r = (S)4 * r * ra - a2 * s2 * ((S)2 * r - (S)2 * M);
  const R Tst = T * dSig_t;
  // alpha^2 = 1 - 2 M r / S2, beta^r = 2 M r / S2
  const R e = M * iS2 * iS2, ialpha = rS2 * g1;
  const R a1 = ((S)2 * r2 - Sig) * e, b1 = Tst * r * e;
  d->alpha[0] = Rr * a1 * ialpha;
  d->alpha[1] = b1 * ialpha;
  d->beta1[0] = (S)-2 * a1 - dxi * f->c.beta1;
  d->beta1[1] = (S)-2 * b1 * iR;
  // h^11 = A / (Sigma S2 R^2)
  const R dls = (S)2 * r * iSig;
  d->l11[0] = Rr * (dA_r * iA - dls - (S)2 * (r + M) * iS2) - (S)2 * dxi;
  d->l11[1] = Tst * (Del * iA - iSig - iS2);  // dA/dtheta = Del dSigma/dtheta
  d->z[0] = Rr * dls;
  d->z[1] = Tst * iSig;
  d->ct = (S)2 * T * c * s * is2;
  if constexpr (kMap) d->tt = (S)2 * p.dtd * T * p.itd2;
  else d->tt = R((S)0);
}

// Coordinate velocity of a particle at a point: v1 = alpha u^1 / gamma -
// beta^1, v2 = alpha u^2 / gamma, w3 = alpha u^3 / gamma.  With p = u_1 / R and
// D = S2 (m^2 Sigma + u_2^2 / T^2 + 2 a p u_3 + u_3^2 / sin^2) + A p^2, the
// closed forms of App. A give alpha / gamma = Sigma / sqrt(D), and Sigma cancels:
//   v1 = ((A p + a u_3 S2) / sqrt(D) - 2 M r) / (R S2),  v2 = u_2 / (T^2 sqrt(D)),
//   w3 = (a p + u_3 / sin^2) / sqrt(D):
// one reciprocal and one inverse square root, and none of the six coefficients.
// The push is bound by vector instructions; with this, the frame of three
// inverse square roots below, the logarithmic derivatives of the force, the
// anchors and the scalar constants of the series, ten steps and a sort went
// from 4569 to 4017 us (512^2, 16 per cell, double precision), 76.6 to 65.5 ms
// (1024^2, 90 per cell, double) and 62 to 59.1 ms (2048^2, 32 per cell, single).
template <class R>
struct VelT {
  R v1, v2, w3;
};

// D grows like r^4 gamma^2, which leaves the range of single precision at gamma
// r^2 = 1.8e19.  The velocity stays the same when u and m are scaled alike, so
// for ultrarelativistic particles single precision multiplies them first by the
// power of two (exact) of ig, 1 / gamma or an estimate: then the range is that of
// gamma^2, as in the other stages.  (For every particle: 1 % of a full step at
// 2048^2 with 32 per cell; this way 0.3 %.)  In double precision D has room for
// gamma r^2 = 1e154.
template <class R>
__device__ inline void scale_momenta(R ig, R& u1, R& u2, R& u3, R& mass2) {
  if constexpr (sizeof(R) == 4) {
    if (ig < 0x1p-20f) {
      const int e = __builtin_amdgcn_frexp_expf(ig);
      u1 = ldexpf(u1, e);
      u2 = ldexpf(u2, e);
      u3 = ldexpf(u3, e);
      mass2 = ldexpf(mass2, 2 * e);
    }
  }
}

template <class R>
__device__ inline VelT<R> velocity_from(const Grid& g, RSCT<R> p, Scalar<R> u1, Scalar<R> u2, Scalar<R> u3,
                                        Scalar<R> mass2) {
  const R r = p.r, s = p.s, c = p.c, Rr = p.rd;
  using S = Scalar<R>;
  const UniT<S> U = uni<R>(g);
  const S a = U.a, a2 = U.a2, au3 = a * u3;
  const R r2 = r * r;
  const R tMr = U.two_M * r;
  const R Sig = r2 + a2 * c * c;
  const R S2 = Sig + tMr;
  const R ra = r2 + a2;
  const R s2 = s * s;
  const R A = ra * ra - a2 * (ra - tMr) * s2;
  const R x = S2 * s2;
  const R q = rcp(Rr * x);
  const R iR = x * q, y = Rr * q;  // y = 1 / (S2 sin^2)
  const R iS2 = s2 * y, is2 = S2 * y;
  const R p1 = u1 * iR, t3 = u3 * is2;
  const R Ap = A * p1;
  const R B = mass2 * Sig + (u2 * u2) * p.itd2 + ((S)2 * au3) * p1 + u3 * t3;
  const R gi = rsqrt(S2 * B + Ap * p1);
  VelT<R> v;
  v.v1 = iR * iS2 * ((Ap + au3 * S2) * gi - tMr);
  v.v2 = p.itd2 * u2 * gi;
  v.w3 = (a * p1 + t3) * gi;
  return v;
}

// Geometry at a grid location for the field solver (theta not clamped).
struct Cell {
  double alpha, beta1, hl11, hl22, hl33, hl13;
  double sqrt_h, sqrt_ht;  // sqrt(h) and sqrt(h) / sin(theta)
};

__host__ __device__ inline Cell cell_at(const Grid& g, double x1, double x2) {
  double r, R, th, T, dT;
  map_r(g, x1, &r, &R);
  map_theta(g, x2, &th, &T, &dT);
  double s, c;
  sin_cos(th, &s, &c);
  const double a2 = g.a * g.a, r2 = r * r, tMr = 2.0 * g.M * r;
  const double Sig = r2 + a2 * c * c;
  const double S2 = Sig + tMr;
  const double ra = r2 + a2;
  const double A = ra * ra - a2 * (ra - tMr) * s * s;
  const double iSig = 1.0 / Sig;
  const double opz = S2 * iSig;  // 1 + z
  Cell e;
  e.alpha = sqrt(Sig / S2);
  e.beta1 = tMr / (S2 * R);
  e.hl11 = opz * R * R;
  e.hl22 = Sig * T * T;
  e.hl33 = A * s * s * iSig;
  e.hl13 = -g.a * opz * s * s * R;
  e.sqrt_ht = R * T * Sig / e.alpha;
  e.sqrt_h = e.sqrt_ht * s;
  return e;
}

// gamma = sqrt(m^2 + h^ij u_i u_j) (Sec. 2.3; mass2 = 1 massive, 0 massless)
__host__ __device__ inline double gamma_of(const Coeffs& m, double u1, double u2, double u3,
                                           double mass2 = 1.0) {
  return sqrt(mass2 + m.hu11 * u1 * u1 + m.hu22 * u2 * u2 + m.hu33 * u3 * u3 +
              2.0 * m.hu13 * u1 * u3);
}

}  // namespace grpic
