// particles.hpp -- push and deposit kernels, FP64 form and single-precision form.
//
// One particle per lane; structure-of-arrays loads and stores are contiguous
// across a wavefront.  The push follows Sec. 3.1 steps 1-11 of the paper; the
// deposit Sec. 3.2.  The single-precision form stores cell indices as int32
// and offsets, momenta, fields and currents as float, evaluates the metric in
// float from offsets relative to the particle's cell (angles from the nearer
// axis), and takes the metric and its derivatives at x^n in FP64 inside the
// horizon region (cells i1 < i_fp64).
#pragma once

#include <type_traits>

#include <climits>

#include "geometry.hpp"

namespace grpic {

constexpr uint8_t kLeaving = 0x80;
constexpr uint8_t kInvalid = 0x40;  // dropped by a bounds guard; never used again
constexpr uint8_t kSpecies = 0x03;
constexpr uint8_t kMassless = 0x04;  // with species 3: a massless neutral particle

__host__ __device__ inline bool is_live(uint8_t t) { return t != 0 && !(t & kInvalid); }

// m^2 in gamma = sqrt(m^2 + h^ij u_i u_j) (Sec. 2.3): 0 for a massless neutral
// particle (species 3 with the massless bit), 1 otherwise
__host__ __device__ inline double mass2_of(uint8_t t) {
  return (t & (kSpecies | kMassless)) == (kSpecies | kMassless) ? 0.0 : 1.0;
}

// a position inside the grid (what the push may start from)
template <class T>
__device__ inline bool in_grid(const Grid& g, int i1, T dx1, int i2, T dx2) {
  // (no short-circuit: a branch per term would make each array's load wait
  // for the one before it)
  return (i1 >= 0) & (i1 < g.n_r) & (i2 >= 0) & (i2 < g.n_th) & (dx1 >= (T)0) & (dx1 <= (T)1) &
         (dx2 >= (T)0) & (dx2 <= (T)1);
}

// a position the deposit may write around: one cell beyond the radial edges
template <class T>
__device__ inline bool in_deposit_range(const Grid& g, int i1, T dx1, int i2, T dx2) {
  return (i1 >= -1) & (i1 <= g.n_r) & (i2 >= 0) & (i2 < g.n_th) & (dx1 >= (T)0) & (dx1 <= (T)1) &
         (dx2 >= (T)0) & (dx2 <= (T)1);
}

template <class T>
struct ParticleArraysT {
  int32_t* __restrict__ i1;
  int32_t* __restrict__ i2;
  T* __restrict__ dx1;
  T* __restrict__ dx2;
  T* __restrict__ u1;
  T* __restrict__ u2;
  T* __restrict__ u3;
  T* __restrict__ w;
  T* __restrict__ phi;
  int32_t* __restrict__ i1p;
  int32_t* __restrict__ i2p;
  T* __restrict__ dx1p;
  T* __restrict__ dx2p;
  uint8_t* __restrict__ tag;
  int64_t n;
};
using ParticleArrays = ParticleArraysT<double>;

template <class T>
struct GatherPlanesT {
  const T* __restrict__ D[3];
  const T* __restrict__ B[3];
};

template <class T = double>
__device__ inline T species_sign(uint8_t t) {
  const int s = t & kSpecies;
  return s == 1 ? (T)1 : (s == 2 ? (T)-1 : (T)0);
}

// The arrays from slot k0 on (a block's first slot: uniform), so that a lane
// reaches its slot with a 32-bit index.
template <class T>
__device__ inline ParticleArraysT<T> from_slot(const ParticleArraysT<T>& P, int64_t k0) {
  return ParticleArraysT<T>{P.i1 + k0, P.i2 + k0, P.dx1 + k0, P.dx2 + k0, P.u1 + k0, P.u2 + k0, P.u3 + k0,
                            P.w + k0, P.phi + k0, P.i1p + k0, P.i2p + k0, P.dx1p + k0, P.dx2p + k0, P.tag + k0, P.n - k0};
}

// The block of slots that a block of the double-precision fused pass takes.
// Block b runs on XCD b mod 8.  In a cell-sorted set the blocks beside the axes,
// which take the longer form of the polar terms, recur with the length of a
// theta row; where that is a multiple of 8 blocks, slot block b on block b gives
// them all to one or two XCDs, and the others wait.  So each XCD takes 64 slot
// blocks in a row of every group of 512; the last, partial group keeps its
// order.  512^2 with 16 per cell (rows of 64 blocks), ten whole steps: 3.37 to
// 3.12 ms; 1024^2 with 90 per cell (rows of 720): 58.47 and 58.47 ms.  Runs of 16
// gave 3.23 and 60.2 ms, of 256 3.15 and 60.3 (60.3 without).  Turning the place
// of an XCD from group to group cost 1 % at 1024^2, and the single-precision
// pass, whose polar terms differ less near the axes, gains nothing from either
// (0 to -1 %).
__device__ inline int64_t spread_block() {
  const unsigned b = blockIdx.x;
  if ((b | 511u) >= gridDim.x) return b;
  return (int64_t)((b & ~511u) | ((b & 7u) << 6) | ((b >> 3) & 63u));
}

// First-order interpolation in code coordinates of the six field components
// (D^1, D^2, D^3, B^1, B^2, B^3) at offsets (dx1, dx2) in cell (i1, i2); a
// component staggered by half a cell starts at the cell's corner or one row or
// column before it.  O: uint32_t byte offsets where g.narrow says they hold (the
// planes' bases and the second row's are then scalar), int64_t otherwise.
template <class O, class T>
__device__ inline void gather_off(const Grid& g, const GatherPlanesT<T>& fp, int i1, T dx1, int i2, T dx2, T F[6]) {
  const T half = (T)0.5;
  const bool up1 = dx1 >= half, up2 = dx2 >= half;
  const T h1 = up1 ? dx1 - half : dx1 + half, h2 = up2 ? dx2 - half : dx2 + half;
  O o;
  if constexpr (sizeof(O) == 4) o = ((O)__umul24((unsigned)(i1 + g.ng), (unsigned)g.ld) + (O)(i2 + g.ng)) * (O)sizeof(T);
  else o = (O)ix(g, i1, i2) * (O)sizeof(T);
  const O row = (O)g.ld * (O)sizeof(T);
  const O oa = up1 ? o : o - row, ob = up2 ? o : o - (O)sizeof(T), oab = up2 ? oa : oa - (O)sizeof(T);
  auto at = [&](const T* __restrict__ p, O off, T w1, T w2) {
    const T* a = (const T*)((const char*)p + (size_t)off);
    const T* b = (const T*)((const char*)p + (size_t)row + (size_t)off);
    const T f00 = a[0], f01 = a[1], f10 = b[0], f11 = b[1];
    const T a0 = f00 + w2 * (f01 - f00);
    const T a1 = f10 + w2 * (f11 - f10);
    return a0 + w1 * (a1 - a0);
  };
  F[0] = at(fp.D[0], oa, h1, dx2);
  F[1] = at(fp.D[1], ob, dx1, h2);
  F[2] = at(fp.D[2], o, dx1, dx2);
  F[3] = at(fp.B[0], ob, dx1, h2);
  F[4] = at(fp.B[1], oa, h1, dx2);
  F[5] = at(fp.B[2], oab, h1, h2);
}
template <class T>
__device__ inline void gather(const Grid& g, const GatherPlanesT<T>& fp, int i1, T dx1, int i2, T dx2, T F[6]) {
  if (g.narrow) gather_off<uint32_t>(g, fp, i1, dx1, i2, dx2, F);
  else gather_off<int64_t>(g, fp, i1, dx1, i2, dx2, F);
}

// Relativistic Boris step for duration tau in an orthonormal frame: u_minus
// = u + k E, the rotation (u_minus + u_minus x t) x s, the second electric
// half kick.  Returns the change of u (both kicks plus the rotation term).
template <class R>
__device__ inline void boris_delta(R ux, R uy, R uz, const R E[3], const R B[3], R k /* = qm tau / 2 */,
                                   R& dx, R& dy, R& dz) {
  // (single precision: reciprocal and reciprocal square root from the
  // hardware seeds with a Newton step, about an ulp, in place of the
  // correctly rounded division and square root)
  const R mx = ux + k * E[0], my = uy + k * E[1], mz = uz + k * E[2];
  const R ig = k * rsqrt((R)1 + mx * mx + my * my + mz * mz);
  const R tx = B[0] * ig, ty = B[1] * ig, tz = B[2] * ig;
  const R f = (R)2 * rcp((R)1 + tx * tx + ty * ty + tz * tz);
  const R sx = f * tx, sy = f * ty, sz = f * tz;
  const R px = mx + (my * tz - mz * ty);
  const R py = my + (mz * tx - mx * tz);
  const R pz = mz + (mx * ty - my * tx);
  const R k2 = k + k;
  dx = (py * sz - pz * sy) + k2 * E[0];
  dy = (pz * sx - px * sz) + k2 * E[1];
  dz = (px * sy - py * sx) + k2 * E[2];
}

// The same Boris step applied to u in place (reciprocal and reciprocal square
// root as in boris_delta; in double precision seeds with one third-order step,
// about an ulp).
template <class R>
__device__ inline void boris(R& ux, R& uy, R& uz, const R E[3], const R B[3], R k /* = qm tau / 2 */) {
  const R mx = ux + k * E[0], my = uy + k * E[1], mz = uz + k * E[2];
  const R ig = k * rsqrt((R)1 + mx * mx + my * my + mz * mz);
  const R tx = B[0] * ig, ty = B[1] * ig, tz = B[2] * ig;
  const R f = (R)2 * rcp((R)1 + tx * tx + ty * ty + tz * tz);
  const R sx = f * tx, sy = f * ty, sz = f * tz;
  const R px = mx + (my * tz - mz * ty);
  const R py = my + (mz * tx - mx * tz);
  const R pz = mz + (mx * ty - my * tx);
  ux = mx + (py * sz - pz * sy) + k * E[0];
  uy = my + (pz * sx - px * sz) + k * E[1];
  uz = mz + (px * sy - py * sx) + k * E[2];
}

// EM half step: covariant -> tetrad (App. A), Boris, tetrad -> covariant:
// u_hat1 = u^1 / sqrt(h^11), u_hat2 = u_2 / sqrt(h_22), u_hat3 = u_3 / sqrt(h_33).
// Single precision takes only the change of the tetrad components back and
// adds it to the covariant u, so u carries one rounding per half step instead
// of those of a full round trip through the tetrad (which would dominate the
// error of the single-precision form over many steps).  Double precision
// takes the whole vector back: the round trip costs nothing visible there, and
// it keeps fewer values live.
template <class R>
__device__ inline void em_half(const FrameT<R>& f, const R E[3], const R B[3], R k, R& u1, R& u2,
                               R& u3) {
  const R k13 = f.c.hu13 * f.is11;
  if constexpr (sizeof(R) == 4) {
    const R x = f.is11 * (f.c.hu11 * u1 + f.c.hu13 * u3);
    const R y = u2 * (f.c.hu22 * f.s22);
    const R z = u3 * f.is33;
    R dx, dy, dz;
    boris_delta(x, y, z, E, B, k, dx, dy, dz);
    const R d3 = f.s33 * dz;
    u1 = u1 + f.is11 * (dx - k13 * d3);
    u2 = u2 + f.s22 * dy;
    u3 = u3 + d3;
  } else {
    R x = f.is11 * (f.c.hu11 * u1 + f.c.hu13 * u3);
    R y = u2 * (f.c.hu22 * f.s22);
    R z = u3 * f.is33;
    boris(x, y, z, E, B, k);
    u3 = f.s33 * z;
    u1 = f.is11 * (x - k13 * u3);
    u2 = f.s22 * y;
  }
}

// Implicit-midpoint geodesic momentum update at fixed x^n (eq.
// discretized-geodesic-u); u_3 is untouched.  With t_jk the terms h^jk b_j b_k
// of gamma^2, the force's sum over the metric derivatives is one over the
// logarithmic derivatives times those terms (GradT).
// kMap: the general map (GradT::tt is not 0).
template <bool kMap, bool kCycle, class R>
__device__ inline void geodesic_u(const Grid& g, const FrameT<R>& f, const GradT<R>& d, R& u1, R& u2,
                                  R u3, R mass2) {
  const CoeffsT<R>& m = f.c;
  const R s1 = u1, s2 = u2;
  const R t33 = m.hu33 * u3 * u3, c13 = (R)2 * m.hu13 * u3, ha = (R)0.5 * m.alpha;
  const R ct33 = d.ct * t33;
  const R dt = uni<R>(g).dt, dxi = uni<R>(g).dxi;
  R t1 = s1, t2 = s2;
  R o1 = (R)__builtin_nan(""), o2 = o1;  // the iterate before t (none yet)
  for (int it = 0; it < g.n_iter; ++it) {
    const R b1 = (R)0.5 * (s1 + t1), b2 = (R)0.5 * (s2 + t2);
    const R t11 = m.hu11 * b1 * b1, t22 = m.hu22 * b2 * b2, t13 = c13 * b1;
    const R W = t22 + t13 + t33;
    const R Q = mass2 + t11 + W;
    const R ig = rsqrt(Q);
    const R gb = Q * ig, h = ha * ig;
    const R q1 = d.l11[0] * t11 - d.z[0] * W - dxi * t13;
    R q2 = d.l11[1] * t11 - d.z[1] * W - ct33;
    if (kMap) q2 = q2 - d.tt * t22;
    const R n1 = s1 + dt * (b1 * d.beta1[0] - gb * d.alpha[0] - h * q1);
    const R n2 = s2 + dt * (b1 * d.beta1[1] - gb * d.alpha[1] - h * q2);
    // exact repeat: the fixed point of the map; kCycle: an iterate that equals
    // the one before the last: from here on the two alternate, and the last of
    // the n_iter is this one or its predecessor by parity; or the optional
    // convergence test, evaluated in FP64
    const bool cycle = kCycle && n1 == o1 && n2 == o2;
    if (cycle && ((g.n_iter - it) & 1) == 0) break;
    bool fixed = cycle || (n1 == t1 && n2 == t2);
    if (g.iter_tol > 0.0)
      fixed = fixed || fabs((double)n1 - (double)t1) + fabs((double)n2 - (double)t2) <=
                           g.iter_tol * (fabs((double)n1) + fabs((double)n2));
    o1 = t1;
    o2 = t2;
    t1 = n1;
    t2 = n2;
    if (fixed) break;
  }
  u1 = t1;
  u2 = t2;
}

template <class R>
__device__ inline void renormalize(int& i, R& dx) {
  const R f = floor(dx);
  i += (int)f;
  dx -= f;
  if (dx >= (R)1) {
    dx -= (R)1;
    i += 1;
  }
}

// exp(t) for |t| <= 0.11: Taylor series to t^11 (remainder below 1e-20 relative)
__device__ inline double exp_small(double t) {
  double p = fma_k(t, 1.0 / 39916800.0, 1.0 / 3628800.0);
  p = fma_k(t, p, 1.0 / 362880.0);
  p = fma_k(t, p, 1.0 / 40320.0);
  p = fma_k(t, p, 1.0 / 5040.0);
  p = fma_k(t, p, 1.0 / 720.0);
  p = fma_k(t, p, 1.0 / 120.0);
  p = fma_k(t, p, 1.0 / 24.0);
  p = fma_k(t, p, 1.0 / 6.0);
  p = fma(t, p, 0.5);
  p = fma(t, p, 1.0);
  return fma(t, p, 1.0);
}

// sin and cos for |x| <= 0.11: Taylor series to x^13 and x^14
__device__ inline void sincos_small(double x, double* s, double* c) {
  const double z = x * x;
  double ps = fma_k(z, 1.0 / 6227020800.0, -1.0 / 39916800.0);
  ps = fma_k(z, ps, 1.0 / 362880.0);
  ps = fma_k(z, ps, -1.0 / 5040.0);
  ps = fma_k(z, ps, 1.0 / 120.0);
  ps = fma_k(z, ps, -1.0 / 6.0);
  *s = fma(x * z, ps, x);
  double pc = fma_k(z, -1.0 / 87178291200.0, 1.0 / 479001600.0);
  pc = fma_k(z, pc, -1.0 / 3628800.0);
  pc = fma_k(z, pc, 1.0 / 40320.0);
  pc = fma_k(z, pc, -1.0 / 720.0);
  pc = fma_k(z, pc, 1.0 / 24.0);
  pc = fma(z, pc, -0.5);
  *c = fma(z, pc, 1.0);
}

// exp(t) for |t| <= 0.03: Taylor series to t^8 (remainder below 1e-19 relative)
__device__ inline double exp_short(double t) {
  double p = fma_k(t, 1.0 / 40320.0, 1.0 / 5040.0);
  p = fma_k(t, p, 1.0 / 720.0);
  p = fma_k(t, p, 1.0 / 120.0);
  p = fma_k(t, p, 1.0 / 24.0);
  p = fma_k(t, p, 1.0 / 6.0);
  p = fma(t, p, 0.5);
  p = fma(t, p, 1.0);
  return fma(t, p, 1.0);
}

// sin and cos for |x| <= 0.03: Taylor series to x^7 and x^6 (remainders
// below 2e-17 relative)
__device__ inline void sincos_short(double x, double* s, double* c) {
  const double z = x * x;
  double ps = fma_k(z, -1.0 / 5040.0, 1.0 / 120.0);
  ps = fma_k(z, ps, -1.0 / 6.0);
  *s = fma(x * z, ps, x);
  double pc = fma_k(z, -1.0 / 720.0, 1.0 / 24.0);
  pc = fma(z, pc, -0.5);
  *c = fma(z, pc, 1.0);
}

// Forms of the position's r, sin and cos (the SER of the kernels below): 0 the
// library functions; 1, 2 the long and the short series on the logarithmic-r,
// uniform-theta grid; 3 the short series on the general quasi-spherical map, in
// double precision only (701 x 533, 24 per cell, ten steps with the fused pass:
// 8.5 -> 7.3 ms; in single precision, where the library functions are short
// and the horizon cells take the other, 4.26 -> 4.31 ms).
constexpr bool is_map(int ser) { return ser == 0 || ser == 3; }

// The general map next to node eta = i2 dth: theta(eta + d) - theta(eta) =
// d (q0 + q1 d + 2 c d^2) and T / dth = q0 + 2 q1 d + 6 c d^2, c = 2 h0 / pi^2,
// q0 = T / dth at the node, q1 = c (6 eta - 3 pi).
template <class R>
struct MapNodeT {
  R q0, q1;
};

// pi - (pi rounded to double)
constexpr double kPiLo = 1.2246467991473531772e-16;

// r, sin and cos at code position (x1, x2) near cell (i1, i2) on the
// logarithmic-r, uniform-theta grid, as rsc_at below has them for the cells next
// to an axis (rsc_horizon; SER = 0: the library functions on any grid).
template <int SER>
__device__ inline RSC rsc_near(const Grid& g, const Tables& t, int i1, double x1, int i2, double x2) {
  if (SER == 0) return rsc_direct(g, x1, x2);
  RSC p;
  const double tr = (x1 - (double)i1) * g.dxi;
  p.r = t.r[0][i1 + g.ng] * (SER == 2 ? exp_short(tr) : exp_small(tr));
  p.rd = g.dxi * p.r;
  p.td = g.dth;
  p.itd2 = g.inv_dth2;
  p.dtd = 0.0;
  const double th = x2 * g.dth;
  const double band = SER == 2 ? g.axis_band : 0.11;
  if (th <= g.small_angle) {
    p.s = g.sin_lo;
    p.c = g.cos_lo;
  } else if (th >= g.th_hi) {
    p.s = g.sin_hi;
    p.c = g.cos_hi;
  } else if (th <= band) {
    if (SER == 2) sincos_short(th, &p.s, &p.c); else sincos_small(th, &p.s, &p.c);
  } else if (th >= (SER == 2 ? g.band_hi : kPi - 0.11)) {
    double cq;
    if (SER == 2) sincos_short((kPi - th) + kPiLo, &p.s, &cq);
    else sincos_small((kPi - th) + kPiLo, &p.s, &cq);
    p.c = -cq;
  } else {
    double sp, cp;
    if (SER == 2) sincos_short(th - (double)i2 * g.dth, &sp, &cp);
    else sincos_small(th - (double)i2 * g.dth, &sp, &cp);
    const double sj = t.s[0][i2 + g.ng], cj = t.c[0][i2 + g.ng];
    p.s = fma(sj, cp, cj * sp);
    p.c = fma(cj, cp, -(sj * sp));
  }
  return p;
}

// single-precision series for |x| <= 0.11 (truncation below 1e-9 relative)
__device__ inline float exp_small_f(float t) {
  float p = fmaf(t, 1.0f / 720.0f, 1.0f / 120.0f);
  p = fmaf(t, p, 1.0f / 24.0f);
  p = fmaf(t, p, 1.0f / 6.0f);
  p = fmaf(t, p, 0.5f);
  p = fmaf(t, p, 1.0f);
  return fmaf(t, p, 1.0f);
}

__device__ inline void sincos_small_f(float x, float* s, float* c) {
  const float z = x * x;
  float ps = fmaf(z, -1.0f / 5040.0f, 1.0f / 120.0f);
  ps = fmaf(z, ps, -1.0f / 6.0f);
  *s = fmaf(x * z, ps, x);
  float pc = fmaf(z, 1.0f / 40320.0f, -1.0f / 720.0f);
  pc = fmaf(z, pc, 1.0f / 24.0f);
  pc = fmaf(z, pc, -0.5f);
  *c = fmaf(z, pc, 1.0f);
}

// Single precision: r, sin, cos and the map factors at offsets (f1, f2) from
// the corner of cell (i1, i2), |f| <= 1.5.  The polar angle is measured from
// the nearer axis, theta(x2) or pi - theta(x2) = theta(n_th - x2) (the map is
// symmetric about the equator), so that sin keeps its relative precision next
// to either axis; clamped at small_angle.  SER > 0: the logarithmic-r,
// uniform-theta grid with series; SER = 0: the general map of App. A with the
// library functions.
template <int SER>
__device__ inline RSCT<float> rsc_near_f(const Grid& g, const Tables& t, int i1, float f1, int i2,
                                        float f2) {
  RSCT<float> p;
  const float dth = g.uf.dth, eps = g.uf.small_angle;
  const float e = elem(t.rf, (uint32_t)(i1 + g.ng)) * (SER > 0 ? exp_small_f(f1 * g.uf.dxi) : expf(f1 * g.uf.dxi));
  p.r = SER > 0 ? e : (float)g.r0 + e;
  p.rd = g.uf.dxi * e;
  const bool upper = 2 * i2 >= g.n_th;
  const float eta = upper ? ((float)(g.n_th - i2) - f2) * dth : ((float)i2 + f2) * dth;
  float ang = eta;
  if (SER > 0) {
    p.td = dth;
    p.itd2 = g.uf.inv_dth2;
    p.dtd = 0.0f;
  } else {
    // past the axis (a midpoint of the coordinate iteration) the map is
    // continued by reflection, as in map_theta: theta odd, T even, dT odd
    const bool past = eta < 0.0f;
    const float ea = past ? -eta : eta;
    const float h0 = (float)g.h0, pi = (float)kPi, y = ea * (float)(1.0 / kPi);
    const float th = ea + 2.0f * h0 * ea * (pi - 2.0f * ea) * (pi - ea) * (float)(1.0 / (kPi * kPi));
    ang = past ? -th : th;
    p.td = dth * (1.0f + 2.0f * h0 + 12.0f * h0 * y * (y - 1.0f));
    p.itd2 = rcp(p.td * p.td);
    const float dd = dth * dth * 12.0f * h0 * (2.0f * y - 1.0f) * (float)(1.0 / kPi);
    p.dtd = (upper != past) ? -dd : dd;
  }
  float s, c;
  if (ang <= eps) {
    s = (float)g.sin_lo;
    c = (float)g.cos_lo;
  } else if (SER == 0) {
    sincosf(ang, &s, &c);
  } else if (ang <= 0.11f) {
    sincos_small_f(ang, &s, &c);
  } else {
    // angle addition about the table node theta_i2 (float tables)
    float sp, cp;
    sincos_small_f(f2 * dth, &sp, &cp);
    const float sj = t.sf[i2 + g.ng], cj = t.cf[i2 + g.ng];
    p.s = fmaf(sj, cp, cj * sp);
    p.c = fmaf(cj, cp, -(sj * sp));
    return p;
  }
  p.s = s;
  p.c = upper ? -c : c;
  return p;
}

// The tables' values at a cell's corner, read once per particle: positions in
// the cells at least mid64 / mid32 from both axes (mid) need nothing else, and
// the iterations of the coordinate update then neither read memory nor branch on
// the angle.  The form depends on the particle's cell alone, so a result does not
// depend on the other lanes.  In double precision the lanes beside an axis that
// are outside its band share the table form with those of other cells: a
// wavefront with both then runs two forms, not three (separate push, 512^2 with 16
// per cell: 264 -> 242 us).
template <class T>
struct AnchorT {
  T r, s, c;       // r - r0; sin, cos
  MapNodeT<T> q;   // general map
  bool mid;
};

// Whether column i2 is at least m cells from both axes.
__device__ inline bool in_middle(const Grid& g, int m, int i2) { return i2 >= m && i2 < g.n_th - m; }

template <int SER>
__device__ inline AnchorT<double> anchor_at(const Grid& g, const Tables& t, int i1, int i2, double) {
  AnchorT<double> a;
  a.mid = false;
  if (SER > 0) {
    a.r = elem(t.r[0], (uint32_t)(i1 + g.ng));
    a.s = elem(t.s[0], (uint32_t)(i2 + g.ng));
    a.c = elem(t.c[0], (uint32_t)(i2 + g.ng));
    if (SER == 3) {
      a.r -= g.r0;
      a.q.q0 = elem(t.td[0], (uint32_t)(i2 + g.ng)) * g.inv_dth;
      a.q.q1 = 12.0 * g.h0 * (1.0 / (kPi * kPi)) * ((double)i2 * g.dth - 0.5 * kPi);
    }
    a.mid = in_middle(g, g.mid64, i2);
  }
  return a;
}
template <int SER>
__device__ inline AnchorT<float> anchor_at(const Grid& g, const Tables& t, int i1, int i2, float) {
  AnchorT<float> a;
  a.mid = false;
  if (SER > 0) {
    a.r = elem(t.rf, (uint32_t)(i1 + g.ng));
    a.s = elem(t.sf, (uint32_t)(i2 + g.ng));
    a.c = elem(t.cf, (uint32_t)(i2 + g.ng));
    a.mid = in_middle(g, g.mid32, i2);
  }
  return a;
}

// The same as rsc_at below for the horizon cells of the single-precision push
// (r0 = 0 where SER > 0), whose kernels have no registers to keep an anchor
// through the axis form (spilled, a ranked pass takes 10 % longer).
template <int SER>
__device__ inline RSC rsc_horizon(const Grid& g, const Tables& t, const AnchorT<double>& an, int i1, double x1, double f1,
                                  int i2, double x2, double f2) {
  if (SER == 0 || !an.mid) return rsc_near<SER>(g, t, i1, x1, i2, x2);
  RSC p;
  const double tr = f1 * g.dxi;
  double sp, cp;
  const double x = f2 * g.dth;
  p.td = g.dth;
  p.itd2 = g.inv_dth2;
  p.dtd = 0.0;
  if (SER == 1) sincos_small(x, &sp, &cp); else sincos_short(x, &sp, &cp);
  p.r = an.r * (SER == 1 ? exp_small(tr) : exp_short(tr));
  p.rd = g.dxi * p.r;
  p.s = fma(an.s, cp, an.c * sp);
  p.c = fma(an.c, cp, -(an.s * sp));
  return p;
}

// r, sin, cos and the map factors at offsets (f1, f2) from the corner of cell
// (i1, i2), |f| <= 1.5, position (x1, x2): r = r0 + (r_i - r0) exp(f1 dxi), and the
// polar angle by angle addition from the table node.  Within an axis band, which
// only the cells that are not `mid` can reach, that would cancel: there the angle
// is rounded and clamped as theta = clamp(x2 dth) (or the general map's) first,
// and the result is the sine and cosine of that double, by a series on theta
// itself next to theta = 0, on psi = pi - theta (exact subtraction plus the low
// part of pi) next to theta = pi, so that sin keeps its relative precision.
// SER = 2: offsets |f| dxi, |f| dth <= 0.03 and a band of 4 cells (its angles <=
// 0.03): short series throughout.  SER = 1: offsets <= 0.11 and a band of 0.11
// rad: long series.  SER = 3: the general map on grids whose offsets are within
// 0.03 and whose cells 8 from an axis within 0.11 rad: short series, long ones
// in a band of 0.11 rad.  SER = 0: library functions.
template <int SER>
__device__ inline RSC rsc_at(const Grid& g, const Tables& t, const AnchorT<double>& an, int i1, double x1, double f1,
                             int i2, double x2, double f2) {
  if (SER == 0) return rsc_direct(g, x1, x2);
  RSC p;
  p.td = g.dth;
  p.itd2 = g.inv_dth2;
  p.dtd = 0.0;
  bool table = an.mid;
  if (!table) {
    double th;
    if (SER == 3) map_theta(g, x2, &th, &p.td, &p.dtd);
    else th = x2 * g.dth;
    const double lo = SER == 2 ? g.axis_band : 0.11, hi = SER == 2 ? g.band_hi : kPi - 0.11;
    table = th > lo && th < hi;
    if (!table) {
      const bool upper = th >= hi;
      const double q = upper ? (kPi - th) + kPiLo : th;
      if (SER == 2) sincos_short(q, &p.s, &p.c); else sincos_small(q, &p.s, &p.c);
      p.c = upper ? -p.c : p.c;
      if (th <= g.small_angle) {
        p.s = g.sin_lo;
        p.c = g.cos_lo;
      } else if (th >= g.th_hi) {
        p.s = g.sin_hi;
        p.c = g.cos_hi;
      }
    }
  }
  if (table) {
    double sp, cp, x = f2 * g.dth;
    if (SER == 3) {
      const double c2 = 4.0 * g.h0 * (1.0 / (kPi * kPi)), d = x, w = c2 * d;  // 2 c
      x = d * (an.q.q0 + d * (an.q.q1 + w));
      p.td = g.dth * (an.q.q0 + d * (2.0 * an.q.q1 + 3.0 * w));
      p.dtd = g.dth * g.dth * (2.0 * an.q.q1 + 6.0 * w);
    }
    if (SER == 1) sincos_small(x, &sp, &cp); else sincos_short(x, &sp, &cp);
    p.s = fma(an.s, cp, an.c * sp);
    p.c = fma(an.c, cp, -(an.s * sp));
  }
  if (SER == 3) {
    const double it = rcp(p.td);
    p.itd2 = it * it;
  }
  const double tr = f1 * g.dxi;
  p.r = an.r * (SER == 1 ? exp_small(tr) : exp_short(tr));
  p.rd = g.dxi * p.r;
  if (SER == 3) p.r += g.r0;
  return p;
}
template <int SER>
__device__ inline RSCT<float> rsc_at(const Grid& g, const Tables& t, const AnchorT<float>& an, int i1, double,
                                     float f1, int i2, double, float f2) {
  if (SER == 0 || !an.mid) return rsc_near_f<SER>(g, t, i1, f1, i2, f2);
  RSCT<float> p;
  float sp, cp;
  sincos_small_f(f2 * g.uf.dth, &sp, &cp);
  p.r = an.r * exp_small_f(f1 * g.uf.dxi);
  p.rd = g.uf.dxi * p.r;
  p.td = g.uf.dth;
  p.itd2 = g.uf.inv_dth2;
  p.dtd = 0.0f;
  p.s = fmaf(an.s, cp, an.c * sp);
  p.c = fmaf(an.c, cp, -(an.s * sp));
  return p;
}

// Whether a move is of one cell at most, which is what the deposit's footprint
// holds.  A displacement below one cell is not enough: an offset of 1, which
// in_grid accepts and a reflection at an axis can leave, plus the largest number
// below 1 rounds to 2.
__host__ __device__ inline bool one_cell_move(int ia, int ja, int ib, int jb) {
  return (unsigned)(ib - ia + 1) <= 2u && (unsigned)(jb - ja + 1) <= 2u;
}

// Sort key of a slot's state: its cell i1 * n_th + i2, or n_cells for a slot
// that the cell sort drops (empty, invalid, leaving, outside the grid).
__device__ inline int cell_key(const Grid& g, uint8_t t, int i1, int i2) {
  if (!is_live(t) || (t & kLeaving) || i1 < 0 || i1 >= g.n_r || i2 < 0 || i2 >= g.n_th) return g.n_r * g.n_th;
  return i1 * g.n_th + i2;
}

// The state a push starts from, its eight loads issued together: behind a
// branch on the tag, and one per term of the bounds check, they would be five
// memory latencies one after the other in every wavefront (ten steps and a
// sort: 4096^2 with 16 per cell in single precision 141.1 -> 132.1 ms, 1024^2
// with 90 per cell in double precision 81.7 -> 76.6 ms).
template <class T>
struct StateT {
  uint8_t t;
  int i1, i2;
  T dx1, dx2, u1, u2, u3;
};

template <class T>
__device__ inline StateT<T> load_state(const ParticleArraysT<T>& P, uint32_t k) {
  StateT<T> s;
  s.t = elem(P.tag, k);
  s.i1 = elem(P.i1, k);
  s.i2 = elem(P.i2, k);
  s.dx1 = elem(P.dx1, k);
  s.dx2 = elem(P.dx2, k);
  s.u1 = elem(P.u1, k);
  s.u2 = elem(P.u2, k);
  s.u3 = elem(P.u3, k);
  // (the empty asm keeps the compiler from moving a load down to its first use)
  uint32_t t = s.t;
  asm volatile("" : "+v"(t), "+v"(s.i1), "+v"(s.i2), "+v"(s.dx1), "+v"(s.dx2), "+v"(s.u1), "+v"(s.u2), "+v"(s.u3));
  s.t = (uint8_t)t;
  return s;
}

// What the deposit needs from one particle's move (Sec. 3.2).
template <class T>
struct Move {
  bool dep;            // deposits a current this step
  bool mid;            // vphi holds alpha u^3 / gamma at the deposit's path midpoint
  int ia, ja, ib, jb;  // previous and current cell
  T xa, ya, xb, yb;    // previous and current offsets
  T q;                 // species sign x charge_scale x weight
  T vphi;
  T u1, u2, u3;        // u^{n+1/2}, for vphi when !mid
  int cell;            // sort key of the state after the push (cell_key)
};

// Implicit coordinate update (eq. discretized-geodesic-x): the displacement
// (d1, d2) in cells and w3, the phi velocity alpha u^3 / gamma at the path
// midpoint.  An iterate that repeats exactly is the fixed point of the map, so
// stopping there gives the same result as running all n_iter iterations (and
// with iter_tol > 0 the loop also ends once the FP64 change is below the
// relative tolerance).  Rounding may end the iteration in two values that
// alternate instead: with kCycle an iterate equal to the one before the last
// decides the remaining ones, and the loop ends with what n_iter iterations give.
// The first iterate (d = 0) uses the coefficients m at
// x^n already in hand; w3 is that of the last evaluation if the iterate
// repeats there, and of one more at the final midpoint otherwise.
template <int SER, bool kCycle, class R>
__device__ inline void coordinate_update(const Grid& g, const Tables& tab, const AnchorT<R>& an, const CoeffsT<R>& m,
                                         int i1, R dx1, int i2, R dx2, R u1, R u2, R u3, R mass2, R& d1, R& d2,
                                         R& w3) {
  const R dt = uni<R>(g).dt, half = (R)0.5;
  const R ig = rsqrt(mass2 + m.hu11 * u1 * u1 + m.hu22 * u2 * u2 + m.hu33 * u3 * u3 + (R)2 * m.hu13 * u1 * u3);
  const R iu0 = m.alpha * ig;
  R n1 = dt * ((m.hu11 * u1 + m.hu13 * u3) * iu0 - m.beta1);
  R n2 = dt * (m.hu22 * u2 * iu0);
  w3 = (m.hu13 * u1 + m.hu33 * u3) * iu0;
  d1 = (R)0;
  d2 = (R)0;
  scale_momenta(ig, u1, u2, u3, mass2);
  R o1 = (R)__builtin_nan(""), o2 = o1;  // the iterate before d (none yet)
  for (int it = 1;; ++it) {
    const bool repeat = n1 == d1 && n2 == d2, cycle = kCycle && n1 == o1 && n2 == o2;
    if (cycle && ((g.n_iter - it) & 1)) break;  // (d, w3) is where they end
    bool last = cycle || it >= g.n_iter;
    if (g.iter_tol > 0.0)
      last = last || fabs((double)n1 - (double)d1) + fabs((double)n2 - (double)d2) <=
                         g.iter_tol * (fabs((double)n1) + fabs((double)n2));
    o1 = d1;
    o2 = d2;
    d1 = n1;
    d2 = n2;
    if (repeat) break;
    const VelT<R> v = velocity_from(g,
                                    rsc_at<SER>(g, tab, an, i1, ((double)i1 + (double)dx1) + 0.5 * (double)d1,
                                                dx1 + half * d1, i2, ((double)i2 + (double)dx2) + 0.5 * (double)d2,
                                                dx2 + half * d2),
                                    u1, u2, u3, mass2);
    w3 = v.w3;
    if (last) break;
    n1 = dt * v.v1;
    n2 = dt * v.v2;
  }
}

// FP64 particle update (Sec. 3.1 steps 1-11) of slot k of the block's arrays
// (from_slot); writes the new state
// and returns the move for the deposit.
template <int SER, bool kPrev = true, bool kCycle = false>
__device__ inline Move<double> push_one(const Grid& g, const Tables& tab, const GatherPlanesT<double>& fp,
                                        const ParticleArrays& P, uint32_t k) {
  Move<double> mv;
  mv.dep = false;
  mv.cell = g.n_r * g.n_th;
  if ((int64_t)k >= P.n) return mv;
  const StateT<double> st = load_state(P, k);
  uint8_t t = st.t;
  if (!is_live(t)) return mv;
  if (t & kLeaving) {
    elem(P.tag, k) = 0;
    return mv;
  }
  int i1 = st.i1, i2 = st.i2;
  double dx1 = st.dx1, dx2 = st.dx2;
  if (!in_grid(g, i1, dx1, i2, dx2)) {  // corrupt input: drop, never index with it
    elem(P.tag, k) = kInvalid;
    return mv;
  }
  double u1 = st.u1, u2 = st.u2, u3 = st.u3;
  if (kPrev) {  // the previous position, for a separate deposit
    elem(P.i1p, k) = i1;
    elem(P.i2p, k) = i2;
    elem(P.dx1p, k) = dx1;
    elem(P.dx2p, k) = dx2;
  }
  mv.ia = i1;
  mv.ja = i2;
  mv.xa = dx1;
  mv.ya = dx2;

  AnchorT<double> an = anchor_at<SER>(g, tab, i1, i2, 0.0);
  Frame f;
  Grad d;
  frame_from<is_map(SER)>(g, rsc_at<SER>(g, tab, an, i1, (double)i1 + dx1, dx1, i2, (double)i2 + dx2, dx2), &f, &d);
  const double qm = species_sign(t);
  if (qm != 0.0) {
    // D^i, B^i at x^n -> tetrad components, scaled by the lapse
    double F[6];
    gather(g, fp, i1, dx1, i2, dx2, F);
    const double al = f.c.alpha, ais11 = al * f.is11, k13 = f.c.hu13 * f.is11 * f.is11;
    const double E[3] = {ais11 * F[0], al * f.s22 * F[1], al * f.s33 * (F[2] - k13 * F[0])};
    const double B[3] = {ais11 * F[3], al * f.s22 * F[4], al * f.s33 * (F[5] - k13 * F[3])};
    const double kb = 0.25 * qm * g.dt;
    em_half(f, E, B, kb, u1, u2, u3);
    geodesic_u<is_map(SER), kCycle>(g, f, d, u1, u2, u3, 1.0);
    em_half(f, E, B, kb, u1, u2, u3);
  } else {
    geodesic_u<is_map(SER), kCycle>(g, f, d, u1, u2, u3, mass2_of(t));  // EM stage skipped for q = 0
  }

  // m^2 and the anchor, taken here again rather than kept from the top: the
  // empty asm keeps the compiler from hoisting them, so that they are not live
  // through the field gather and EM stages, where the FP64 update is at its
  // register limit
  uint32_t tl = t;
  asm volatile("" : "+v"(tl), "+v"(i1), "+v"(i2));
  an = anchor_at<SER>(g, tab, i1, i2, 0.0);
  const double ms = mass2_of((uint8_t)tl);
  // the weight and phi, needed after the iterations: in flight during them
  const double wt = elem(P.w, k), ph = elem(P.phi, k);
  double d1, d2, w3;
  coordinate_update<SER, kCycle>(g, tab, an, f.c, i1, dx1, i2, dx2, u1, u2, u3, ms, d1, d2, w3);
  elem(P.phi, k) = ph + g.dt * w3;
  mv.vphi = w3;
  dx1 += d1;
  renormalize(i1, dx1);
  dx2 += d2;
  renormalize(i2, dx2);
  mv.mid = true;
  if (i2 < 0) {
    i2 = 0;
    dx2 = 1.0 - dx2;
    u2 = -u2;
    mv.mid = false;
  } else if (i2 >= g.n_th) {
    i2 = g.n_th - 1;
    dx2 = 1.0 - dx2;
    u2 = -u2;
    mv.mid = false;
  }
  if (i1 < 0 || i1 >= g.n_r) t |= kLeaving;
  // a non-finite or more-than-one-cell move cannot be deposited: drop it
  if (!(fabs(d1) < 1.0 && fabs(d2) < 1.0)) t = kInvalid;
  elem(P.i1, k) = i1;
  elem(P.i2, k) = i2;
  elem(P.dx1, k) = dx1;
  elem(P.dx2, k) = dx2;
  elem(P.u1, k) = u1;
  elem(P.u2, k) = u2;
  elem(P.u3, k) = u3;
  elem(P.tag, k) = t;
  mv.dep = is_live(t) && qm != 0.0 && one_cell_move(mv.ia, mv.ja, i1, i2);
  mv.ib = i1;
  mv.jb = i2;
  mv.xb = dx1;
  mv.yb = dx2;
  mv.q = (qm * g.charge_scale) * wt;
  mv.u1 = u1;
  mv.u2 = u2;
  mv.u3 = u3;
  mv.cell = cell_key(g, t, i1, i2);
  return mv;
}

// Single-precision form of the same update (see the file comment).
template <int SER, bool kPrev = true>
__device__ inline Move<float> push_one_f32(const Grid& g, const Tables& tab, const GatherPlanesT<float>& fp,
                                           const ParticleArraysT<float>& P, uint32_t k) {
  Move<float> mv;
  mv.dep = false;
  mv.cell = g.n_r * g.n_th;
  if ((int64_t)k >= P.n) return mv;
  const StateT<float> st = load_state(P, k);
  uint8_t t = st.t;
  if (!is_live(t)) return mv;
  if (t & kLeaving) {
    elem(P.tag, k) = 0;
    return mv;
  }
  int i1 = st.i1, i2 = st.i2;
  float dx1 = st.dx1, dx2 = st.dx2;
  if (!in_grid(g, i1, dx1, i2, dx2)) {
    elem(P.tag, k) = kInvalid;
    return mv;
  }
  float u1 = st.u1, u2 = st.u2, u3 = st.u3;
  if (kPrev) {  // the previous position, for a separate deposit
    elem(P.i1p, k) = i1;
    elem(P.i2p, k) = i2;
    elem(P.dx1p, k) = dx1;
    elem(P.dx2p, k) = dx2;
  }
  mv.ia = i1;
  mv.ja = i2;
  mv.xa = dx1;
  mv.ya = dx2;

  AnchorT<float> an = anchor_at<SER>(g, tab, i1, i2, 0.0f);
  FrameT<float> f;
  GradT<float> d;
  if (i1 < g.i_fp64) {
    // horizon region: metric and derivatives in FP64, then rounded
    Frame fd;
    Grad dd;
    const AnchorT<double> ad = anchor_at<SER>(g, tab, i1, i2, 0.0);
    frame_from<is_map(SER)>(g, rsc_horizon<SER>(g, tab, ad, i1, (double)i1 + dx1, (double)dx1, i2, (double)i2 + dx2, (double)dx2),
                         &fd, &dd);
    f.c = CoeffsT<float>{(float)fd.c.alpha, (float)fd.c.beta1, (float)fd.c.hu11,
                         (float)fd.c.hu22, (float)fd.c.hu33, (float)fd.c.hu13};
    f.is11 = (float)fd.is11;
    f.s22 = (float)fd.s22;
    f.s33 = (float)fd.s33;
    f.is33 = (float)fd.is33;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      d.alpha[q] = (float)dd.alpha[q];
      d.beta1[q] = (float)dd.beta1[q];
      d.l11[q] = (float)dd.l11[q];
      d.z[q] = (float)dd.z[q];
    }
    d.ct = (float)dd.ct;
    d.tt = (float)dd.tt;
  } else {
    frame_from<is_map(SER)>(g, rsc_at<SER>(g, tab, an, i1, 0.0, dx1, i2, 0.0, dx2), &f, &d);
  }
  const float qm = species_sign<float>(t);
  const float ms = (float)mass2_of(t);
  if (qm != 0.0f) {
    float F[6];
    gather(g, fp, i1, dx1, i2, dx2, F);
    const float al = f.c.alpha, ais11 = al * f.is11, k13 = f.c.hu13 * f.is11 * f.is11;
    const float E[3] = {ais11 * F[0], al * f.s22 * F[1], al * f.s33 * (F[2] - k13 * F[0])};
    const float B[3] = {ais11 * F[3], al * f.s22 * F[4], al * f.s33 * (F[5] - k13 * F[3])};
    const float kb = 0.25f * qm * g.uf.dt;
    em_half(f, E, B, kb, u1, u2, u3);
    geodesic_u<is_map(SER), false>(g, f, d, u1, u2, u3, 1.0f);
    em_half(f, E, B, kb, u1, u2, u3);
  } else {
    geodesic_u<is_map(SER), false>(g, f, d, u1, u2, u3, ms);  // EM stage skipped for q = 0
  }

  // the weight and phi, needed after the iterations: in flight during them
  const float wt = elem(P.w, k), ph = elem(P.phi, k);
  float d1, d2;
  asm volatile("" : "+v"(i1), "+v"(i2));  // (the anchor again, as in push_one)
  an = anchor_at<SER>(g, tab, i1, i2, 0.0f);
  coordinate_update<SER, false>(g, tab, an, f.c, i1, dx1, i2, dx2, u1, u2, u3, ms, d1, d2, mv.vphi);
  elem(P.phi, k) = ph + g.uf.dt * mv.vphi;
  dx1 += d1;
  renormalize(i1, dx1);
  dx2 += d2;
  renormalize(i2, dx2);
  mv.mid = true;
  if (i2 < 0) {
    i2 = 0;
    dx2 = 1.0f - dx2;
    u2 = -u2;
    mv.mid = false;
  } else if (i2 >= g.n_th) {
    i2 = g.n_th - 1;
    dx2 = 1.0f - dx2;
    u2 = -u2;
    mv.mid = false;
  }
  if (i1 < 0 || i1 >= g.n_r) t |= kLeaving;
  if (!(fabsf(d1) < 1.0f && fabsf(d2) < 1.0f)) t = kInvalid;
  elem(P.i1, k) = i1;
  elem(P.i2, k) = i2;
  elem(P.dx1, k) = dx1;
  elem(P.dx2, k) = dx2;
  elem(P.u1, k) = u1;
  elem(P.u2, k) = u2;
  elem(P.u3, k) = u3;
  elem(P.tag, k) = t;
  mv.dep = is_live(t) && qm != 0.0f && one_cell_move(mv.ia, mv.ja, i1, i2);
  mv.ib = i1;
  mv.jb = i2;
  mv.xb = dx1;
  mv.yb = dx2;
  mv.q = (qm * g.uf.charge_scale) * wt;
  mv.u1 = u1;
  mv.u2 = u2;
  mv.u3 = u3;
  mv.cell = cell_key(g, t, i1, i2);
  return mv;
}

// The move of slot k as stored by the push (previous and current position).
template <class T>
__device__ inline Move<T> load_move(const Grid& g, const ParticleArraysT<T>& P, uint32_t k) {
  Move<T> mv;
  mv.dep = false;
  mv.mid = false;
  mv.cell = g.n_r * g.n_th;
  if ((int64_t)k >= P.n) return mv;
  const uint8_t t = elem(P.tag, k);
  if (!is_live(t)) return mv;
  const T sg = species_sign<T>(t);
  if (sg == (T)0) return mv;
  mv.dep = true;
  mv.q = (sg * uni<T>(g).charge_scale) * elem(P.w, k);
  mv.ia = elem(P.i1p, k);
  mv.ja = elem(P.i2p, k);
  mv.xa = elem(P.dx1p, k);
  mv.ya = elem(P.dx2p, k);
  mv.ib = elem(P.i1, k);
  mv.jb = elem(P.i2, k);
  mv.xb = elem(P.dx1, k);
  mv.yb = elem(P.dx2, k);
  mv.u1 = elem(P.u1, k);
  mv.u2 = elem(P.u2, k);
  mv.u3 = elem(P.u3, k);
  return mv;
}

template <class T>
struct CurrentPlanesT {
  T* __restrict__ J[3];
};
using CurrentPlanes = CurrentPlanesT<double>;

__device__ inline void atomic_add(double* p, double v) { unsafeAtomicAdd(p, v); }
__device__ inline void atomic_add(float* p, float v) { unsafeAtomicAdd(p, v); }

// ------------------------------------------------------------------ deposit
// Charge-conserving zigzag split (Sec. 3.2) of the move from (ia + xa, ja + ya)
// to (ib + xb, jb + yb): the path is cut at the relay point r, each segment
// deposits J^1 and J^2 (normalised by 1/dt) on the edges of the cell it lies
// in, with first-order weights at the segment midpoint; J^3 = q alpha u^3 /
// gamma goes to the four nodes around the path midpoint.
// Particles per block of the deposit passes (two wavefronts).  Blocks of 64 in
// single precision: +1.6 % (2048^2, 16 per cell).
constexpr int kDepBlock = 128;

// The LDS tile around the block's anchor cell has kTilePlane nodes per
// component, laid out as 1 << LC columns: 8 rows of 16 in two copies, between
// which the adding lanes alternate (a cell's run of lanes then hits one address
// with half of its lanes per copy), 8 rows of 32, or 4 of 64.  It holds the
// footprints of cells up to kI rows and kJ - 1 columns from the anchor.
constexpr int kTilePlane = 2 * kDepBlock;
template <int LC>
struct TileT {
  static constexpr int kC = 1 << LC, kRows = LC == 6 ? 4 : 8, kRep = kTilePlane / (kC * kRows);
  static constexpr int kI = kRows / 2 - 1, kJ = kC / 2 - 1;  // the anchor cell's row and column
};

// Sets of at least kDenseSlots slots per cell take the tile of 16 columns: 128
// cell-sorted slots then span 12 cells at most, of the 13 that it holds.  Below,
// every block takes its tile by the columns that its particles span (kSparse; 0:
// no tile).  Fused pass at 1024^2 in single precision, just sorted / after ten
// steps without a sort, us, with 16 columns and by the span: 16 per cell 450 /
// 459 and 456 / 473; 12 345 / 381 and 354 / 377; 10 299 / 380 and 299 / 321; 6 408
// / 542 and 194 / 212; 4 347 / 457 and 156 / 201; 2 214 / 285 and 84 / 208; in double
// precision 12 637 / 648 and 658 / 642; 10 556 / 552 and 559 / 552; 6 439 / 561 and
// 363 / 361; 2 241 / 319 and 141 / 249.
constexpr int kDenseSlots = 11;
inline bool is_sparse(const Grid& g, int64_t n) { return n < (int64_t)kDenseSlots * g.n_r * g.n_th; }
__device__ inline int tile_columns(int span) { return span <= 40 ? 5 : span <= 160 ? 6 : 0; }

// lapse-weighted phi velocity alpha u^3 / gamma at the path midpoint (ia + xm, ja + ym)
template <int SER, class T>
__device__ inline T vphi_mid(const Grid& g, const Tables& tab, int ia, T xm, int ja, T ym, T u1, T u2, T u3) {
  T mass2 = (T)1;
  if constexpr (sizeof(T) == 4)  // an estimate of 1 / gamma, up to factors of r and the cell sizes
    scale_momenta(rcp(fmaxf(fmaxf(fabsf(u1), fabsf(u2)), fmaxf(fabsf(u3), mass2))), u1, u2, u3, mass2);
  const AnchorT<T> an = anchor_at<SER>(g, tab, ia, ja, (T)0);
  return velocity_from(g, rsc_at<SER>(g, tab, an, ia, (double)ia + (double)xm, xm, ja, (double)ja + (double)ym, ym), u1,
                       u2, u3, mass2).w3;
}

// The nodes and weights of one move: footprint [ia-1, ia+2] x [ja-1, ja+2].
template <class T>
struct ContribT {
  int di, dj, km, lm;     // cell step, J^3 node corner (relative to (ia, ja))
  T j1[4], j2[4], j3[4];  // J^1 at (ia, ja), (ia, ja+1), (ib, jb), (ib, jb+1); J^2 at (ia, ja), (ia+1, ja),
                          // (ib, jb), (ib+1, jb); J^3 at (km, lm), (km, lm+1), (km+1, lm), (km+1, lm+1)
};

// A stored move that the zigzag can represent: both ends in range, a cell at
// most apart.  (The moves of a fused pass are: the push starts inside the grid,
// reflects at the axes and deposits one_cell_move only.)
template <class T>
__device__ inline bool move_in_range(const Grid& g, const Move<T>& mv) {
  const bool from = in_grid(g, mv.ia, mv.xa, mv.ja, mv.ya), to = in_deposit_range(g, mv.ib, mv.xb, mv.jb, mv.yb);
  return from & to & one_cell_move(mv.ia, mv.ja, mv.ib, mv.jb);
}

template <class T, int SER>
__device__ inline ContribT<T> make_contrib(const Grid& g, const Tables& tab, const Move<T>& mv) {
  ContribT<T> c;
  const int ia = mv.ia, ja = mv.ja;
  const int di = mv.ib - ia, dj = mv.jb - ja;
  const T q = mv.q;
  const T qdt = q * uni<T>(g).inv_dt;
  const T one = (T)1, half = (T)0.5;
  const T xa = mv.xa, ya = mv.ya;
  const T fi = (T)di, fj = (T)dj;
  const T xb = fi + mv.xb, yb = fj + mv.yb;
  const T xm = half * (xa + xb), ym = half * (ya + yb);
  // relay point: the midpoint, clamped to the faces the two cells share
  const T xr = fmin(fmin((T)0, fi) + one, fmax(fmax((T)0, fi), xm));
  const T yr = fmin(fmin((T)0, fj) + one, fmax(fmax((T)0, fj), ym));
  const T fx1 = qdt * (xr - xa), fy1 = qdt * (yr - ya);
  const T fx2 = qdt * (xb - xr), fy2 = qdt * (yb - yr);
  const T wx1 = half * (xa + xr), wy1 = half * (ya + yr);
  const T wx2 = half * (xr + xb) - fi, wy2 = half * (yr + yb) - fj;
  c.di = di;
  c.dj = dj;
  // f (1 - w) as f - f w: the pair sums to f to rounding
  c.j1[1] = fx1 * wy1;
  c.j1[0] = fx1 - c.j1[1];
  c.j1[3] = fx2 * wy2;
  c.j1[2] = fx2 - c.j1[3];
  c.j2[1] = fy1 * wx1;
  c.j2[0] = fy1 - c.j2[1];
  c.j2[3] = fy2 * wx2;
  c.j2[2] = fy2 - c.j2[3];
  const T vphi = mv.mid ? mv.vphi : vphi_mid<SER>(g, tab, ia, xm, ja, ym, mv.u1, mv.u2, mv.u3);
  const T fm = floor(xm), gm = floor(ym);
  const T w1 = xm - fm, w2 = ym - gm;
  const T c3 = q * vphi, p1 = c3 * w1, p0 = c3 - p1;
  c.km = (int)fm;
  c.lm = (int)gm;
  c.j3[1] = p0 * w2;
  c.j3[0] = p0 - c.j3[1];
  c.j3[3] = p1 * w2;
  c.j3[2] = p1 - c.j3[3];
  // The particle's mirror image in the nearer axis (Sec. 3.3.2) adds the same
  // contribution on an axis node row (j = 0 or n_th) with the component's axis
  // parity: J^1 (even) doubles there, J^3 (odd) cancels, so the axis rows hold
  // the two-sided values the polar-cap update takes with 2 pi.  The footprint
  // spans node rows ja - 1 .. ja + 2, so only particles within two rows of an
  // axis can reach one (a wavefront-uniform skip for cell-sorted particles).
  if (ja <= 1 || ja >= g.n_th - 2) {
    auto e1 = [&](int j) { return (j == 0 || j == g.n_th) ? (T)2 : one; };
    auto e3 = [&](int j) { return (j == 0 || j == g.n_th) ? (T)0 : one; };
    c.j1[0] *= e1(ja);
    c.j1[1] *= e1(ja + 1);
    c.j1[2] *= e1(ja + dj);
    c.j1[3] *= e1(ja + dj + 1);
    const T f0 = e3(ja + c.lm), f1 = e3(ja + c.lm + 1);
    c.j3[0] *= f0;
    c.j3[1] *= f1;
    c.j3[2] *= f0;
    c.j3[3] *= f1;
  }
  return c;
}

// Runs of equal keys in consecutive lanes of a wavefront: `end` is the last
// lane of this lane's run, `head` marks the first lane of a run.
struct Runs {
  int end;
  bool head;
};

__device__ inline Runs runs_of(int key) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(key, 1, 64);
  Runs r;
  r.head = lane == 0 || prev != key;
  const unsigned long long heads = __ballot(r.head);
  const unsigned long long after = lane == 63 ? 0ull : (heads >> (lane + 1));
  r.end = after ? lane + __ffsll((long long)after) - 1 : 63;
  return r;
}

// Sum of v over this lane's run from this lane to the run's end (the head
// ends up with the run total): segmented suffix sum by doubling.
template <class T>
__device__ inline T run_sum(T v, const Runs& r) {
  const int lane = threadIdx.x & 63;
  for (int off = 1; off < 64; off <<= 1) {
    const bool more = lane + off <= r.end;
    if (!__any(more)) break;  // no run is that long
    const T o = __shfl_down(v, off, 64);
    if (more) v += o;
  }
  return v;
}

// The value of the other lane of an aligned pair (2k <-> 2k+1) by DPP quad
// permutation (a VALU move, no LDS traffic); `off` if that lane is inactive.
__device__ inline int pair_swap(int v, int off) {
  return __builtin_amdgcn_update_dpp(off, v, 0xB1, 0xF, 0xF, false);
}
__device__ inline float pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ inline double pair_swap(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

// Block barrier for data in LDS only: a __syncthreads also waits for the
// wavefront's global stores and atomics (here the particle state just written)
// to complete, and the passes' barriers order nothing but LDS.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The cell a block's tile is laid around: that of a live particle in the
// middle of the block's slots (cell-sorted: near the middle of its cells), the
// first of their second half or else the last of the first.  span: the columns
// from the block's first live particle to its last (the shorter way where the
// cells wrap from the end of one theta row to the next).  The slots are kChunks
// chunks of two wavefronts; ia, ja: the cells of a thread's particles.  Every
// thread of the block calls this; false if the block has no live particle.  It
// passes a block barrier.
template <int kChunks>
__device__ inline bool block_anchor(const Grid& g, const bool (&act)[kChunks], const int (&ia)[kChunks],
                                    const int (&ja)[kChunks], int& ai, int& aj, int& span) {
  // of each wavefront's 64 slots: row (INT_MIN: none is live) and column of the particle nearest to the
  // block's middle, column of the one nearest to its ends
  __shared__ int4 cell[2 * kChunks];
  const int wv = (int)threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const unsigned long long live = __ballot(act[c]);
    const int first = (__ffsll((long long)live) - 1) & 63, last = (63 - __clzll((long long)live)) & 63;
    const bool second = 2 * c + wv >= kChunks;
    const int mid = second ? first : last, end = second ? last : first;
    const int wi = __builtin_amdgcn_readlane(ia[c], mid), wj = __builtin_amdgcn_readlane(ja[c], mid);
    const int we = __builtin_amdgcn_readlane(ja[c], end);
    if ((threadIdx.x & 63) == 0) cell[2 * c + wv] = int4{live ? wi : INT_MIN, wj, we, 0};
  }
  lds_barrier();
  int r[2 * kChunks], m[2 * kChunks], x[2 * kChunks];
#pragma unroll
  for (int e = 0; e < 2 * kChunks; ++e) {
    const int4 v = cell[e];
    r[e] = __builtin_amdgcn_readfirstlane(v.x);
    m[e] = __builtin_amdgcn_readfirstlane(v.y);
    x[e] = __builtin_amdgcn_readfirstlane(v.z);
  }
  int from = 0, to = 0;
  ai = INT_MIN;
  aj = 0;
#pragma unroll
  for (int q = 0; q < 2 * kChunks; ++q) {
    const int up = q, down = 2 * kChunks - 1 - q;
    if (r[up] != INT_MIN) to = up < kChunks ? m[up] : x[up];
    if (r[down] != INT_MIN) from = down < kChunks ? x[down] : m[down];
    const int e = q < kChunks ? q : 3 * kChunks - 1 - q;  // the first half upwards, then the second downwards
    if (r[e] != INT_MIN) {
      ai = r[e];
      aj = m[e];
    }
  }
  const int d = abs(from - to);
  span = min(d, g.n_th - d);
  return ai != INT_MIN;
}

// Adds a lane's contributions to the tile, its cell (di, dj) from the anchor;
// false if the footprint leaves the tile.
template <int LC, class T>
__device__ inline bool tile_add(double* tile, int di, int dj, const ContribT<T>& c, const T a[4], const T m[4], bool stay,
                                bool own_a, bool own_m) {
  using L = TileT<LC>;
  const int row = di + L::kI - 1, col = dj + L::kJ - 1;  // the footprint's first row and column
  if ((unsigned)row > (unsigned)(L::kRows - 4) || (unsigned)col > (unsigned)(L::kC - 4)) return false;
  double* t = tile + (row + 1) * L::kC + (col + 1);
  if (L::kRep == 2) t += (threadIdx.x & 2) * (kTilePlane / 4);
  if (own_a) {
    atomicAdd(t, (double)a[0]);
    atomicAdd(t + 1, (double)a[1]);
    atomicAdd(t + kTilePlane, (double)a[2]);
    atomicAdd(t + kTilePlane + L::kC, (double)a[3]);
  }
  if (!stay) {
    double* p = t + c.di * L::kC + c.dj;
    atomicAdd(p, (double)c.j1[2]);
    atomicAdd(p + 1, (double)c.j1[3]);
    atomicAdd(p + kTilePlane, (double)c.j2[2]);
    atomicAdd(p + kTilePlane + L::kC, (double)c.j2[3]);
  }
  if (own_m) {
    double* p = t + 2 * kTilePlane + c.km * L::kC + c.lm;
    atomicAdd(p, (double)m[0]);
    atomicAdd(p + 1, (double)m[1]);
    atomicAdd(p + L::kC, (double)m[2]);
    atomicAdd(p + L::kC + 1, (double)m[3]);
  }
  return true;
}

// Adds the tile to the planes, the copies summed in a fixed order (nodes outside
// the planes are nobody's: their values are zero and never added).
template <int LC, class T>
__device__ inline void tile_flush(const Grid& g, const CurrentPlanesT<T>& cp, const double* tile, int ai, int aj) {
  using L = TileT<LC>;
  constexpr int kNodes = L::kRows * L::kC;
  const int t = (int)threadIdx.x;
  const int64_t base = ix(g, ai - L::kI, aj - L::kJ), off = (int64_t)(t >> LC) * g.ld + (t & (L::kC - 1));
#pragma unroll
  for (int comp = 0; comp < 3; ++comp) {
#pragma unroll
    for (int e = 0; e < kNodes; e += kDepBlock) {
      double val = tile[comp * kTilePlane + e + t];
      if (L::kRep == 2) val += tile[comp * kTilePlane + kNodes + e + t];
      if (val != 0.0) atomic_add(cp.J[comp] + (base + (int64_t)(e / L::kC) * g.ld) + off, (T)val);
    }
  }
}

// Block-level deposit: the lanes add their contributions (12 values, 8 when a
// particle stays in its cell) with LDS atomics to an LDS tile around the
// block's anchor cell; the tile is then added to the planes with one global
// atomic per touched node.  The tile is in double precision in both forms: on gfx950 an
// LDS add of 64 floats takes 194 cycles of the CU even without conflicts, one
// of 64 doubles 9 (21, 93 and 193 with 2, 8 and 64 lanes on one address), and
// the float adds bound the single-precision pass (2048^2, 16 per cell, ten
// steps with the filter and a sort: 30.0 ms, with double adds 26.0).  Before
// the LDS atomics the two lanes of an aligned pair
// that share their nodes are summed by DPP swaps, and only the first adds
// (cell-sorted particles put runs of one cell in consecutive lanes).  A
// particle whose footprint leaves the tile (its block's cells wrap from the end
// of one theta row to the next, or the slots have lost their cell order) adds
// straight to the planes.  The anchor takes the place of a reduction of the
// block's footprint (four wavefront minima and a round trip through LDS), and
// the wider tiles that of a second form with run sums over lanes for whole blocks that
// do not fit.
// (ten steps and a sort: 512^2 with 16 per cell in double precision 3832 ->
// 3574 us, 2048^2 with 32 in single 57.2 -> 54.3 ms; without the flush 2 %,
// without any deposit 6 % (single) to 10 % (double) less.)
// Every lane of the block calls this; it passes a block barrier.
template <class T, int SER, bool kSparse>
__device__ inline void deposit_block(const Grid& g, const Tables& tab, const CurrentPlanesT<T>& cp, const Move<T>& mv,
                                     bool act) {
  constexpr int kBlk = kDepBlock, kPlane = kTilePlane;
  __shared__ __align__(16) double tile[3][kPlane];
  {  // zero the tile (16-byte stores)
    double2* fv = reinterpret_cast<double2*>(&tile[0][0]);
    static_assert(3 * kPlane % (2 * kBlk) == 0, "whole stores per thread");
#pragma unroll
    for (int e = 0; e < 3 * kPlane / 2; e += kBlk) fv[e + (int)threadIdx.x] = double2{};
  }
  int ai, aj, span;
  if (!block_anchor<1>(g, {act}, {mv.ia}, {mv.ja}, ai, aj, span)) return;  // no live charged particle (uniform)
  const int lc = kSparse ? tile_columns(span) : 4;  // (uniform)
  double* const t = &tile[0][0];
  if (act) {
    const ContribT<T> c = make_contrib<T, SER>(g, tab, mv);
    const bool stay = (c.di | c.dj) == 0;
    T a[4] = {c.j1[0], c.j1[1], c.j2[0], c.j2[1]};
    if (stay) {
      a[0] += c.j1[2];
      a[1] += c.j1[3];
      a[2] += c.j2[2];
      a[3] += c.j2[3];
    }
    T m[4] = {c.j3[0], c.j3[1], c.j3[2], c.j3[3]};
    // whether the pair's lanes share their cell, and the J^3 corner too
    const int corner = c.km * 16 + c.lm;
    const int oi = pair_swap(mv.ia, -1), oj = pair_swap(mv.ja, -1), oc = pair_swap(corner, INT_MIN);
    const bool fa = (oi == mv.ia) & (oj == mv.ja), fm = fa & (oc == corner);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const T sa = a[q] + pair_swap(a[q]), sm = m[q] + pair_swap(m[q]);
      a[q] = fa ? sa : a[q];
      m[q] = fm ? sm : m[q];
    }
    const bool second = (threadIdx.x & 1) != 0;
    const bool own_a = !(fa & second), own_m = !(fm & second);
    const int di = mv.ia - ai, dj = mv.ja - aj;
    bool in = false;
    if constexpr (!kSparse) in = tile_add<4>(t, di, dj, c, a, m, stay, own_a, own_m);
    else if (lc == 5) in = tile_add<5>(t, di, dj, c, a, m, stay, own_a, own_m);
    else if (lc == 6) in = tile_add<6>(t, di, dj, c, a, m, stay, own_a, own_m);
    if (!in) {
      const int64_t o = ix(g, mv.ia, mv.ja), ld = g.ld;
      if (own_a) {
        atomic_add(cp.J[0] + o, a[0]);
        atomic_add(cp.J[0] + o + 1, a[1]);
        atomic_add(cp.J[1] + o, a[2]);
        atomic_add(cp.J[1] + o + ld, a[3]);
      }
      if (!stay) {
        const int64_t b = o + c.di * ld + c.dj;
        atomic_add(cp.J[0] + b, c.j1[2]);
        atomic_add(cp.J[0] + b + 1, c.j1[3]);
        atomic_add(cp.J[1] + b, c.j2[2]);
        atomic_add(cp.J[1] + b + ld, c.j2[3]);
      }
      if (own_m) {
        const int64_t n = o + c.km * ld + c.lm;
        atomic_add(cp.J[2] + n, m[0]);
        atomic_add(cp.J[2] + n + 1, m[1]);
        atomic_add(cp.J[2] + n + ld, m[2]);
        atomic_add(cp.J[2] + n + ld + 1, m[3]);
      }
    }
  }
  if (lc == 0) return;
  lds_barrier();
  if (!kSparse) tile_flush<4>(g, cp, t, ai, aj);
  else if (lc == 5) tile_flush<5>(g, cp, t, ai, aj);
  else tile_flush<6>(g, cp, t, ai, aj);
}

// ------------------------------------------------------------------ cell ranks
// The counting sort by cell (cell_key) needs each live slot's rank among the
// slots of its cell and each cell's count.  A block counts its slots per cell
// in an LDS hash table of 2^kBits cells (open addressing, linear probing; at
// most 2^(kBits-1) slots per block, so a free cell is always found): a slot's
// rank inside the block is its cell's count when it was added.  Then one
// returning atomic per cell present in the block claims the block's ranks of
// that cell on the cell's global counter, and every slot takes its cell's
// base plus its rank inside the block.  Slots with key n_cells claim nothing.
template <int kBits>
struct RankTable {
  int key[1 << kBits];
  int n[1 << kBits];  // count in the block, then the cell's base
};

// The block's table (one LDS object per block, whichever function asks).
template <int kBits>
__device__ inline RankTable<kBits>& block_rank_table() {
  __shared__ RankTable<kBits> rt;
  return rt;
}

template <int kBits>
__device__ inline void rank_clear(RankTable<kBits>& rt) {
  for (int e = (int)threadIdx.x; e < (1 << kBits); e += (int)blockDim.x) {
    rt.key[e] = -1;
    rt.n[e] = 0;
  }
}

// Adds a slot of cell `key` (< n_cells) to the table; returns its entry, and
// in `local` the number of the block's slots of that cell added before it.
template <int kBits>
__device__ inline int rank_insert(RankTable<kBits>& rt, int key, int& local) {
  int h = (int)(((uint32_t)key * 0x9E3779B1u) >> (32 - kBits));  // multiplicative hash
  for (;;) {
    const int old = atomicCAS(&rt.key[h], -1, key);
    if (old == -1 || old == key) break;
    h = (h + 1) & ((1 << kBits) - 1);
  }
  local = atomicAdd(&rt.n[h], 1);
  return h;
}

// The claims: afterwards rt.n holds each present cell's base.  Every thread
// of the block calls this after a barrier that follows the last insert (all
// of a thread's claims are in flight before the first is waited for).
template <int kBits, int kThreads>
__device__ inline void rank_claim(RankTable<kBits>& rt, int* __restrict__ counts) {
  constexpr int kE = (1 << kBits) / kThreads;
  int base[kE];
#pragma unroll
  for (int e = 0; e < kE; ++e) {
    const int h = e * kThreads + (int)threadIdx.x;
    const int key = rt.key[h];
    base[e] = key >= 0 ? atomicAdd(counts + key, rt.n[h]) : 0;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kE; ++e) rt.n[e * kThreads + (int)threadIdx.x] = base[e];
  __syncthreads();
}

// Table bits for the slots of a fused block: twice as many cells as slots.
constexpr int kPushRankBits = 8;
static_assert((1 << (kPushRankBits - 1)) >= kDepBlock, "rank table too small");

// The rank pass of the sort inside a fused push + deposit block: slot k's key
// after the push is `cell`; its rank goes to i1p (the previous position is not
// stored by the fused pass).  The table was cleared at the start of the
// kernel and a block barrier (the deposit's) has passed since.
__device__ inline void rank_fused(const Grid& g, int* __restrict__ i1p, uint32_t k, int cell,
                                  int* __restrict__ counts) {
  constexpr int kBits = kPushRankBits;
  RankTable<kBits>& rt = block_rank_table<kBits>();
  int local = 0, entry = -1;
  if (cell < g.n_r * g.n_th) entry = rank_insert(rt, cell, local);
  __syncthreads();
  rank_claim<kBits, kDepBlock>(rt, counts);
  if (entry >= 0) elem(i1p, k) = rt.n[entry] + local;
}

// ------------------------------------------------------------------ kernels
// The FP64 push kernels are held to 128 VGPRs (4 wavefronts per SIMD; the
// series paths of the logarithmic-r, uniform-theta grid do not spill, the general
// map's ranked pass two registers, the library path of the separate push two to
// four): on gfx950 the push is latency- and issue-bound, and the fourth wavefront
// hides more than the compiler's own choice (~160 VGPRs, 3 wavefronts, a 10-15 %
// slower pass); a fifth (96 VGPRs) spills 148 B per lane and runs about 30 %
// slower.
constexpr int kPushBlock = 256;
#define GRPIC_FP64_PUSH_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4)))

// kCycle: the iterations end when two values alternate, for n_iter above
// kCycleIter: up to there the test costs more than the iterations it saves.
// Without / with it, us, 1e6 particles at 256^2 (slots in no order): n_iter = 10 89 /
// 95, 17 92 / 100, 30 102 / 106, 60 123 / 109, 200 233 / 150; 512^2 with 16 per cell
// (sorted): 10 228 / 239, 30 247 / 252, 60 278 / 251, 200 435 / 264.
constexpr int kCycleIter = 32;
template <int SER, bool kCycle>
__global__ void __launch_bounds__(kPushBlock) GRPIC_FP64_PUSH_OCCUPANCY
push_kernel(Grid g, Tables tab, GatherPlanesT<double> fp, ParticleArrays P) {
  (void)push_one<SER, true, kCycle>(g, tab, fp, from_slot(P, (int64_t)blockIdx.x * kPushBlock), threadIdx.x);
}

template <int SER>
__global__ void __launch_bounds__(kPushBlock) push_kernel_f32(Grid g, Tables tab, GatherPlanesT<float> fp,
                                                       ParticleArraysT<float> P) {
  (void)push_one_f32<SER>(g, tab, fp, from_slot(P, (int64_t)blockIdx.x * kPushBlock), threadIdx.x);
}

template <class T, int SER, bool kSparse>
__global__ void __launch_bounds__(kDepBlock) deposit_kernel(Grid g, Tables tab, ParticleArraysT<T> P,
                                                            CurrentPlanesT<T> cp) {
  const Move<T> mv = load_move(g, from_slot(P, (int64_t)blockIdx.x * kDepBlock), threadIdx.x);
  deposit_block<T, SER, kSparse>(g, tab, cp, mv, mv.dep && move_in_range(g, mv));
}

// Push and deposit in one pass: the deposit takes the move from registers and
// J^3 from the push's own midpoint metric; the previous position is not
// stored.  kRank: the pass also ranks the slots by their cell after the push
// for the cell sort (rank_fused; counts: the sort's zeroed cell counters).
template <int SER, bool kRank, bool kSparse>
__global__ void __launch_bounds__(kDepBlock) GRPIC_FP64_PUSH_OCCUPANCY
push_deposit_kernel(Grid g, Tables tab, GatherPlanesT<double> fp, ParticleArrays P, CurrentPlanes cp, int* counts) {
  const ParticleArraysT<double> Q = from_slot(P, spread_block() * kDepBlock);
  if constexpr (kRank) rank_clear(block_rank_table<kPushRankBits>());
  const Move<double> mv = push_one<SER, false>(g, tab, fp, Q, threadIdx.x);
  deposit_block<double, SER, kSparse>(g, tab, cp, mv, mv.dep);
  if constexpr (kRank) rank_fused(g, Q.i1p, threadIdx.x, mv.cell, counts);
}

// library path in FP64 (coarse grids): the library exp and sincos and the map
// factors need more registers than the series paths; three wavefronts per SIMD
// leave room for them without spills
template <bool kRank, bool kSparse>
__global__ void __launch_bounds__(kDepBlock) __attribute__((amdgpu_waves_per_eu(3)))
push_deposit_kernel_lib(Grid g, Tables tab, GatherPlanesT<double> fp, ParticleArrays P, CurrentPlanes cp,
                        int* counts) {
  const ParticleArraysT<double> Q = from_slot(P, spread_block() * kDepBlock);
  if constexpr (kRank) rank_clear(block_rank_table<kPushRankBits>());
  const Move<double> mv = push_one<0, false>(g, tab, fp, Q, threadIdx.x);
  deposit_block<double, 0, kSparse>(g, tab, cp, mv, mv.dep);
  if constexpr (kRank) rank_fused(g, Q.i1p, threadIdx.x, mv.cell, counts);
}

template <int SER, bool kRank, bool kSparse>
__device__ inline void push_deposit_f32(const Grid& g, const Tables& tab, const GatherPlanesT<float>& fp,
                                        const ParticleArraysT<float>& P, const CurrentPlanesT<float>& cp,
                                        int* counts) {
  const ParticleArraysT<float> Q = from_slot(P, (int64_t)blockIdx.x * kDepBlock);
  if constexpr (kRank) rank_clear(block_rank_table<kPushRankBits>());
  const Move<float> mv = push_one_f32<SER, false>(g, tab, fp, Q, threadIdx.x);
  deposit_block<float, SER, kSparse>(g, tab, cp, mv, mv.dep);
  if constexpr (kRank) rank_fused(g, Q.i1p, threadIdx.x, mv.cell, counts);
}

// series paths: 6 wavefronts per SIMD (80 VGPRs; the compiler's own allocation
// takes a few more and 5 wavefronts, 1 to 2 % slower at 2048^2 with 16 per cell)
template <int SER, bool kRank, bool kSparse>
__global__ void __launch_bounds__(kDepBlock) __attribute__((amdgpu_waves_per_eu(6))) push_deposit_kernel_f32(Grid g, Tables tab, GatherPlanesT<float> fp,
                                                                     ParticleArraysT<float> P,
                                                                     CurrentPlanesT<float> cp, int* counts) {
  push_deposit_f32<SER, kRank, kSparse>(g, tab, fp, P, cp, counts);
}

// library path (coarse grids and the general quasi-spherical map): at least 5
// wavefronts per SIMD (80 VGPRs and 6 without the rank pass, 81 and 5 with it)
template <bool kRank, bool kSparse>
__global__ void __launch_bounds__(kDepBlock) __attribute__((amdgpu_waves_per_eu(5)))
push_deposit_kernel_f32_lib(Grid g, Tables tab, GatherPlanesT<float> fp, ParticleArraysT<float> P,
                            CurrentPlanesT<float> cp, int* counts) {
  push_deposit_f32<0, kRank, kSparse>(g, tab, fp, P, cp, counts);
}

}  // namespace grpic
