// adjoint.hpp -- adjoint of one particle update in a frozen field (the
// differentiation form).
//
// The state of a particle is s = (x1, x2, u1, u2, u3), x = cell + offset; the
// field is F = B0 F1.  One step s' = Phi(s, B0) is Sec. 3.1 steps 2-10 with
// the axis reflection and removal of Sec. 3.3.3.  For each particle the kernel
// repeats the step from the stored state and takes the vector-Jacobian product
//   gbar(s) = (ds'/ds)^T gbar(s'),   gbar(B0) += (ds'/dB0) . gbar(s')
// backwards through its stages (a bar marks the derivative of the weighted
// output with respect to a value):
//   coordinates: d = dt v(x + d/2, u).  With lambda = (I - dt/2 v_x^T)^-1 ybar,
//                xbar = ybar + dt v_x^T lambda, ubar += dt v_u^T lambda
//   EM half step (em_reverse), twice, with the bars of the tetrad-frame fields
//   momentum:    Z = s + dt f((s + Z)/2, u3; metric).  With lambda =
//                (I - dt/2 f_b^T)^-1 Zbar, sbar = lambda + dt/2 f_b^T lambda,
//                and the bars of u3 and the metric are dt lambda's
//   gather and metric: the bars of the field components, and of the frame and
//                its first derivatives, go back to x1, x2.
// Both implicit stages are differentiated at their fixed points (the implicit-
// function theorem), which an iterate that has stopped changing is taken for
// (at_fixed: rounding can keep an iteration from an exact repeat for ever).  An
// iteration that does not come that far within n_iter (next to the axis the
// contraction can approach 1) is differentiated through n_iter iterations
// instead.  So the result is the derivative of the map of n_iter iterations; a
// context's iter_tol, which lets the push end earlier, is not looked at.
// The metric depends on the position alone: its derivatives are two tangents
// (Tan<2>) of the same code as the push's, with second derivatives from the
// tangents of its analytic first derivatives.
// Six tangents (x, u, B0) carried through the whole step, the former design,
// needed 490 registers and three times the operations, and iterations that
// rounding kept alternating were run to n_iter.  With 1e6 particles at 256^2
// (20 steps forward, replayed and adjoint): 41.9 -> 14.0 ms.  Bound by its
// vector operations at one wavefront per SIMD (362 registers); held to two or
// three wavefronts it spills and takes 15.0 and 19.0 ms.
#pragma once

#include "particles.hpp"
#include "replay.hpp"
#include "tangent.hpp"

namespace grpic {

using T2 = Tan<2>;

// Whether iterate n (after o) is taken for the fixed point: a relative change
// of at most 1e-14, or one of at most 1e-12 that no longer shrinks (rounding);
// `last`: the change before, updated.
__device__ inline bool at_fixed(double n1, double n2, double o1, double o2, double& last) {
  const double ch = fabs(n1 - o1) + fabs(n2 - o2), size = fabs(n1) + fabs(n2);
  const bool ok = ch <= 1e-14 * size || (ch <= 1e-12 * size && ch >= last);
  last = ch;
  return ok;
}

// Tangents in (x1, x2) of r, sin, cos and the map factors p at polar code
// position x2 (a clamped angle is constant, the map factors are not).
__device__ inline RSCT<T2> rsc_tan(const Grid& g, const RSC& p, double x2) {
  double th, td, dtd;
  map_theta(g, x2, &th, &td, &dtd);
  const bool free = th >= g.small_angle && th <= kPi - g.small_angle;
  auto d1 = [](double v, double d) {
    T2 t(v);
    t.d[0] = d;
    return t;
  };
  auto d2 = [](double v, double d) {
    T2 t(v);
    t.d[1] = d;
    return t;
  };
  RSCT<T2> q;
  q.r = d1(p.r, p.rd);
  q.rd = d1(p.rd, g.dxi * p.rd);
  q.s = d2(p.s, free ? p.td * p.c : 0.0);
  q.c = d2(p.c, free ? -p.td * p.s : 0.0);
  q.td = d2(p.td, p.dtd);
  q.itd2 = d2(p.itd2, -2.0 * p.dtd * p.td * p.itd2 * p.itd2);
  q.dtd = d2(p.dtd, 24.0 * g.h0 * g.dth * g.dth * g.dth * (1.0 / (kPi * kPi)));
  return q;
}

// Coordinate velocity and its derivatives in the position (vx[i][j] =
// dv_i/dx_j) and the momentum (vu[i][j] = dv_i/du_j), in the notation of
// velocity_from: with D the argument of its square root, N1 = A p + a u3 S2
// and N3 = a p + u3 / sin^2, dD/du = 2 (N1 / R, S2 u2 / T^2, S2 N3).
__device__ inline void velocity_jac(const Grid& g, const RSC& p, double x2, double u1, double u2, double u3,
                                    double mass2, double v[2], double vx[2][2], double vu[2][3]) {
  const VelT<T2> t = velocity_from(g, rsc_tan(g, p, x2), u1, u2, u3, mass2);
  v[0] = t.v1.v;
  v[1] = t.v2.v;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    vx[0][j] = t.v1.d[j];
    vx[1][j] = t.v2.d[j];
  }
  const double r2 = p.r * p.r, tMr = g.two_M * p.r, s2 = p.s * p.s;
  const double Sig = r2 + g.a2 * p.c * p.c, S2 = Sig + tMr, ra = r2 + g.a2;
  const double A = ra * ra - g.a2 * (ra - tMr) * s2;
  const double iR = rcp(p.rd), iS2 = rcp(S2), is2 = rcp(s2);
  const double p1 = u1 * iR, N1 = A * p1 + g.a * u3 * S2, N3 = g.a * p1 + u3 * is2;
  const double w2 = u2 * p.itd2;
  const double gi = rsqrt(S2 * (mass2 * Sig + u2 * w2 + g.a * p1 * u3 + u3 * N3) + A * p1 * p1);
  const double g3 = -gi * gi * gi;
  const double D[3] = {g3 * iR * N1, g3 * S2 * w2, g3 * S2 * N3};  // d(1/sqrt(D))/du
  const double c1 = iR * iS2;
  vu[0][0] = c1 * (A * iR * gi + N1 * D[0]);
  vu[0][1] = c1 * N1 * D[1];
  vu[0][2] = c1 * (g.a * S2 * gi + N1 * D[2]);
  vu[1][0] = w2 * D[0];
  vu[1][1] = p.itd2 * gi + w2 * D[1];
  vu[1][2] = w2 * D[2];
}

// Bars of the frame's quantities and of its first derivatives.
struct FrameBar {
  double alpha, hu11, hu13, hu22, hu33, is11, s22, s33, is33;
  double da[2], db[2], l11[2], z[2], ct, tt;
};

// Reverse of em_half (double precision): u, the step's input; (g1, g2, g3),
// the bars of its output on entry and of its input on return; Eb, Bb and m
// accumulate the bars of the tetrad-frame fields and the frame.
__device__ inline void em_reverse(const Frame& f, const double E[3], const double B[3], double k, double u1, double u2,
                                  double u3, double& g1, double& g2, double& g3, double Eb[3], double Bb[3],
                                  FrameBar& m) {
  auto dot = [](const double a[3], const double b[3]) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; };
  auto cross = [](const double a[3], const double b[3], double o[3]) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
  };
  const double k13 = f.c.hu13 * f.is11, N = f.c.hu11 * u1 + f.c.hu13 * u3, f22 = f.c.hu22 * f.s22;
  // the Boris step: q = u + k E, t = B k / sqrt(1 + q^2), w = q + q x t,
  // out = q + w x (F t) + k E, F = 2 / (1 + t^2)
  const double q[3] = {f.is11 * N + k * E[0], u2 * f22 + k * E[1], u3 * f.is33 + k * E[2]};
  const double rn = rsqrt(1.0 + dot(q, q)), ig = k * rn;
  const double t[3] = {ig * B[0], ig * B[1], ig * B[2]};
  const double F = 2.0 * rcp(1.0 + dot(t, t));
  const double s[3] = {F * t[0], F * t[1], F * t[2]};
  double c[3];
  cross(q, t, c);
  const double w[3] = {q[0] + c[0], q[1] + c[1], q[2] + c[2]};
  cross(w, s, c);
  const double o[3] = {q[0] + c[0] + k * E[0], q[1] + c[1] + k * E[1], q[2] + c[2] + k * E[2]};
  // tetrad -> covariant: u3 = s33 o3, u1 = is11 (o1 - k13 u3), u2 = s22 o2
  const double v3 = f.s33 * o[2];
  m.is11 += g1 * (o[0] - k13 * v3);
  double k13b = -g1 * f.is11 * v3;
  const double v3b = g3 - g1 * f.is11 * k13;
  m.s22 += g2 * o[1];
  m.s33 += v3b * o[2];
  const double G[3] = {g1 * f.is11, g2 * f.s22, v3b * f.s33};
  // Boris backwards
  double wb[3], sb[3], tb[3], qb[3];
  cross(s, G, wb);
  cross(G, w, sb);
  const double Fb = dot(sb, t);
  cross(wb, q, c);
#pragma unroll
  for (int i = 0; i < 3; ++i) tb[i] = F * sb[i] + c[i] - F * F * Fb * t[i];
  cross(t, wb, c);
  const double igb = dot(B, tb), n = k * rn * rn * rn * igb;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    qb[i] = G[i] + wb[i] + c[i] - n * q[i];
    Bb[i] += ig * tb[i];
    Eb[i] += k * (G[i] + qb[i]);
  }
  // covariant -> tetrad
  m.is11 += qb[0] * N + k13b * f.c.hu13;
  m.hu11 += qb[0] * f.is11 * u1;
  m.hu13 += qb[0] * f.is11 * u3 + k13b * f.is11;
  m.hu22 += qb[1] * u2 * f.s22;
  m.s22 += qb[1] * u2 * f.c.hu22;
  m.is33 += qb[2] * u3;
  g1 = qb[0] * f.is11 * f.c.hu11;
  g2 = qb[1] * f22;
  g3 = qb[2] * f.is33 + qb[0] * f.is11 * f.c.hu13;
}

// One evaluation of the momentum map n = s + dt f((s + Z)/2, u3) (geodesic_u),
// with the same operations.
struct MomentumMap {
  double s1, s2, t33, c13, ct33, ha, mass2;
};
template <bool kMap>
__device__ inline void momentum_map(const Grid& g, const Frame& f, const Grad& d, const MomentumMap& e, double z1,
                                    double z2, double& n1, double& n2) {
  const CoeffsT<double>& m = f.c;
  const double b1 = 0.5 * (e.s1 + z1), b2 = 0.5 * (e.s2 + z2);
  const double t11 = m.hu11 * b1 * b1, t22 = m.hu22 * b2 * b2, t13 = e.c13 * b1;
  const double W = t22 + t13 + e.t33;
  const double Q = e.mass2 + t11 + W;
  const double ig = rsqrt(Q);
  const double gb = Q * ig, h = e.ha * ig;
  const double q1 = d.l11[0] * t11 - d.z[0] * W - g.dxi * t13;
  double q2 = d.l11[1] * t11 - d.z[1] * W - e.ct33;
  if (kMap) q2 = q2 - d.tt * t22;
  n1 = e.s1 + g.dt * (b1 * d.beta1[0] - gb * d.alpha[0] - h * q1);
  n2 = e.s2 + g.dt * (b1 * d.beta1[1] - gb * d.alpha[1] - h * q2);
}

// Reverse of one evaluation of the momentum force f at (b1, b2, u3): (m1, m2),
// the bars of f; b1b, b2b, those of b; u3b and the frame's accumulate.
template <bool kMap>
__device__ inline void force_reverse(const Grid& g, const Frame& f, const Grad& d, const MomentumMap& e, double u3,
                                     double b1, double b2, double m1, double m2, double& b1b, double& b2b, double& u3b,
                                     FrameBar& mb) {
  const CoeffsT<double>& m = f.c;
  const double h1b = m.hu11 * b1, h2b = m.hu22 * b2;
  const double t11 = h1b * b1, t22 = h2b * b2, t13 = e.c13 * b1;
  const double W = t22 + t13 + e.t33, Q = e.mass2 + t11 + W;
  const double ig = rsqrt(Q), gm = Q * ig, h = e.ha * ig;
  const double q1 = d.l11[0] * t11 - d.z[0] * W - g.dxi * t13;
  double q2 = d.l11[1] * t11 - d.z[1] * W - e.ct33;
  if (kMap) q2 = q2 - d.tt * t22;
  mb.db[0] += m1 * b1;
  mb.db[1] += m2 * b1;
  mb.da[0] -= m1 * gm;
  mb.da[1] -= m2 * gm;
  const double hb = -(m1 * q1 + m2 * q2), q1b = -h * m1, q2b = -h * m2;
  mb.alpha += 0.5 * hb * ig;
  const double Qb = 0.5 * ig * (-(m1 * d.alpha[0] + m2 * d.alpha[1]) - hb * h * ig);
  mb.l11[0] += q1b * t11;
  mb.l11[1] += q2b * t11;
  mb.z[0] -= q1b * W;
  mb.z[1] -= q2b * W;
  mb.ct -= q2b * e.t33;
  if (kMap) mb.tt -= q2b * t22;
  const double Wb = Qb - (q1b * d.z[0] + q2b * d.z[1]);
  const double t11b = Qb + q1b * d.l11[0] + q2b * d.l11[1];
  const double t13b = Wb - g.dxi * q1b, t33b = Wb - q2b * d.ct, t22b = kMap ? Wb - q2b * d.tt : Wb;
  mb.hu11 += t11b * b1 * b1;
  mb.hu22 += t22b * b2 * b2;
  mb.hu13 += t13b * 2.0 * b1 * u3;
  mb.hu33 += t33b * u3 * u3;
  u3b += 2.0 * (t13b * m.hu13 * b1 + t33b * m.hu33 * u3);
  b1b = m1 * d.beta1[0] + m2 * d.beta1[1] + 2.0 * t11b * h1b + t13b * e.c13;
  b2b = 2.0 * t22b * h2b;
}

// df_i/db_j of the momentum force.
template <bool kMap>
__device__ inline void force_jac(const Grid& g, const Frame& f, const Grad& d, const MomentumMap& e, double b1, double b2,
                                 double fb[2][2]) {
  const CoeffsT<double>& m = f.c;
  const double h1b = m.hu11 * b1, h2b = m.hu22 * b2;
  const double t11 = h1b * b1, t22 = h2b * b2, t13 = e.c13 * b1;
  const double W = t22 + t13 + e.t33;
  const double ig = rsqrt(e.mass2 + t11 + W), h = e.ha * ig;
  const double gj[2] = {ig * (h1b + 0.5 * e.c13), ig * h2b};  // dgamma/db
  const double q1 = d.l11[0] * t11 - d.z[0] * W - g.dxi * t13;
  double q2 = d.l11[1] * t11 - d.z[1] * W - e.ct33;
  if (kMap) q2 = q2 - d.tt * t22;
  const double q1j[2] = {2.0 * d.l11[0] * h1b - (d.z[0] + g.dxi) * e.c13, -2.0 * d.z[0] * h2b};
  const double q2j[2] = {2.0 * d.l11[1] * h1b - d.z[1] * e.c13, -2.0 * (kMap ? d.z[1] + d.tt : d.z[1]) * h2b};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const double hj = h * ig * gj[j];  // -dh/db
    fb[0][j] = (j == 0 ? d.beta1[0] : 0.0) - gj[j] * d.alpha[0] + hj * q1 - h * q1j[j];
    fb[1][j] = (j == 0 ? d.beta1[1] : 0.0) - gj[j] * d.alpha[1] + hj * q2 - h * q2j[j];
  }
}

// Reverse of the bilinear gather (reading R2): adds the position bars of the
// six components' bars Fb, and their B0 bar for a field F = B0 F1.
__device__ inline void gather_reverse(const Grid& g, const GatherPlanesT<double>& fp, int i1, double dx1, int i2,
                                      double dx2, const double Fb[6], double& x1b, double& x2b, double& fsum) {
  auto at = [&](const double* __restrict__ F, int h1, int h2, double fb) {
    int k1 = i1, k2 = i2;
    double w1 = dx1, w2 = dx2;
    if (h1) {
      const bool up = dx1 >= 0.5;
      k1 = up ? i1 : i1 - 1;
      w1 = up ? dx1 - 0.5 : dx1 + 0.5;
    }
    if (h2) {
      const bool up = dx2 >= 0.5;
      k2 = up ? i2 : i2 - 1;
      w2 = up ? dx2 - 0.5 : dx2 + 0.5;
    }
    const double* p = F + ix(g, k1, k2);
    const double f00 = p[0], f01 = p[1], f10 = p[g.ld], f11 = p[g.ld + 1];
    const double a0 = f00 + w2 * (f01 - f00), a1 = f10 + w2 * (f11 - f10);
    x1b += fb * (a1 - a0);
    x2b += fb * ((f01 - f00) + w1 * ((f11 - f10) - (f01 - f00)));
    fsum += fb * (a0 + w1 * (a1 - a0));
  };
  at(fp.D[0], 1, 0, Fb[0]);
  at(fp.D[1], 0, 1, Fb[1]);
  at(fp.D[2], 0, 0, Fb[2]);
  at(fp.B[0], 0, 1, Fb[3]);
  at(fp.B[1], 1, 0, Fb[4]);
  at(fp.B[2], 1, 1, Fb[5]);
}

// Reverse of the lapse-scaled tetrad components X of a field triple F (push_one:
// X = alpha (is11 F1, s22 F2, s33 (F3 - h^13 is11^2 F1))): Fb from Xb.
__device__ inline void tetrad_reverse(const Frame& f, const double F[3], const double Xb[3], double Fb[3], FrameBar& m) {
  const double al = f.c.alpha, K = f.c.hu13 * f.is11 * f.is11, d3 = F[2] - K * F[0];
  m.alpha += Xb[0] * f.is11 * F[0] + Xb[1] * f.s22 * F[1] + Xb[2] * f.s33 * d3;
  const double Kb = -Xb[2] * al * f.s33 * F[0];
  m.is11 += Xb[0] * al * F[0] + 2.0 * Kb * f.c.hu13 * f.is11;
  m.hu13 += Kb * f.is11 * f.is11;
  m.s22 += Xb[1] * al * F[1];
  m.s33 += Xb[2] * al * d3;
  Fb[0] = al * (Xb[0] * f.is11 - Xb[2] * f.s33 * K);
  Fb[1] = Xb[1] * al * f.s22;
  Fb[2] = Xb[2] * al * f.s33;
}

// One particle: gbar (x1, x2, u1, u2, u3) is replaced by J_s^T gbar and
// gB0 += J_B0 . gbar.
template <int SER>
__device__ inline void adjoint_one(const Grid& g, const Tables& tab, const GatherPlanesT<double>& fp, double inv_B0,
                                   const ParticleArrays& P, uint32_t k, double gbar[5], double& gB0) {
  constexpr bool kMap = is_map(SER);
  const StateT<double> st = load_state(P, k);
  // empty, removed or leaving particles are not moved by the step: identity
  if (!is_live(st.t) || (st.t & kLeaving)) return;
  const int i1 = st.i1, i2 = st.i2;
  const double dx1 = st.dx1, dx2 = st.dx2;
  if (!in_grid(g, i1, dx1, i2, dx2)) return;
  const double x1 = (double)i1 + dx1, x2 = (double)i2 + dx2;
  const double qm = species_sign(st.t), ms = mass2_of(st.t);
  const AnchorT<double> an = anchor_at<SER>(g, tab, i1, i2, 0.0);
  const RSC p = rsc_at<SER>(g, tab, an, i1, x1, dx1, i2, x2, dx2);
  Frame f;
  Grad d;
  frame_from<kMap>(g, p, &f, &d);

  // the step, keeping each stage's input
  const double kb = 0.25 * qm * g.dt;
  double E[3] = {0.0, 0.0, 0.0}, B[3] = {0.0, 0.0, 0.0};
  double a1 = st.u1, a2 = st.u2, a3 = st.u3;
  if (qm != 0.0) {
    double F[6];
    gather(g, fp, i1, dx1, i2, dx2, F);
    const double al = f.c.alpha, K = f.c.hu13 * f.is11 * f.is11;
    E[0] = al * f.is11 * F[0];
    E[1] = al * f.s22 * F[1];
    E[2] = al * f.s33 * (F[2] - K * F[0]);
    B[0] = al * f.is11 * F[3];
    B[1] = al * f.s22 * F[4];
    B[2] = al * f.s33 * (F[5] - K * F[3]);
    em_half(f, E, B, kb, a1, a2, a3);
  }
  MomentumMap e;
  e.s1 = a1;
  e.s2 = a2;
  e.t33 = f.c.hu33 * a3 * a3;
  e.c13 = 2.0 * f.c.hu13 * a3;
  e.ct33 = d.ct * e.t33;
  e.ha = 0.5 * f.c.alpha;
  e.mass2 = ms;
  double z1 = a1, z2 = a2;
  bool fixed_u = false;
  double last = INFINITY;
  for (int it = 0; it < g.n_iter && !fixed_u; ++it) {
    double n1, n2;
    momentum_map<kMap>(g, f, d, e, z1, z2, n1, n2);
    fixed_u = at_fixed(n1, n2, z1, z2, last);
    z1 = n1;
    z2 = n2;
  }
  double w1 = z1, w2 = z2, w3 = a3;
  if (qm != 0.0) em_half(f, E, B, kb, w1, w2, w3);

  // coordinate stage, backwards
  double x1b = gbar[0], x2b = gbar[1], u1b = gbar[2], u2b = gbar[3], u3b = gbar[4];
  {
    double d1 = 0.0, d2 = 0.0;
    bool fixed = false;
    last = INFINITY;
    for (int it = 0; it < g.n_iter && !fixed; ++it) {
      const VelT<double> v =
          velocity_from(g, rsc_at<SER>(g, tab, an, i1, x1 + 0.5 * d1, dx1 + 0.5 * d1, i2, x2 + 0.5 * d2, dx2 + 0.5 * d2),
                        w1, w2, w3, ms);
      const double n1 = g.dt * v.v1, n2 = g.dt * v.v2;
      fixed = at_fixed(n1, n2, d1, d2, last);
      d1 = n1;
      d2 = n2;
    }
    // axis reflection: x2 -> -x2 below theta = 0, 2 n_th - x2 above theta = pi
    const double y2 = floor(x2 + d2);
    if (y2 < 0.0 || y2 >= (double)g.n_th) {
      x2b = -x2b;
      u2b = -u2b;
    }
    double v[2], vx[2][2], vu[2][3];
    if (fixed) {
      const double m1 = x1 + 0.5 * d1, m2 = x2 + 0.5 * d2;
      velocity_jac(g, rsc_at<SER>(g, tab, an, i1, m1, dx1 + 0.5 * d1, i2, m2, dx2 + 0.5 * d2), m2, w1, w2, w3, ms, v, vx,
                   vu);
      const double hd = 0.5 * g.dt;
      const double c11 = 1.0 - hd * vx[0][0], c22 = 1.0 - hd * vx[1][1], c12 = hd * vx[1][0], c21 = hd * vx[0][1];
      const double id = g.dt / (c11 * c22 - c12 * c21);
      const double l1 = (c22 * x1b + c12 * x2b) * id, l2 = (c21 * x1b + c11 * x2b) * id;  // dt lambda
      x1b += vx[0][0] * l1 + vx[1][0] * l2;
      x2b += vx[0][1] * l1 + vx[1][1] * l2;
      u1b += vu[0][0] * l1 + vu[1][0] * l2;
      u2b += vu[0][1] * l1 + vu[1][1] * l2;
      u3b += vu[0][2] * l1 + vu[1][2] * l2;
    } else {
      // M = d(d1, d2)/d(x1, x2, u1, u2, u3) through the n_iter iterations run
      double M[2][5] = {};
      d1 = d2 = 0.0;
      for (int it = 0; it < g.n_iter; ++it) {
        const double m1 = x1 + 0.5 * d1, m2 = x2 + 0.5 * d2;
        velocity_jac(g, rsc_at<SER>(g, tab, an, i1, m1, dx1 + 0.5 * d1, i2, m2, dx2 + 0.5 * d2), m2, w1, w2, w3, ms, v,
                     vx, vu);
#pragma unroll
        for (int j = 0; j < 5; ++j) {
          const double p1 = (j == 0 ? 1.0 : 0.0) + 0.5 * M[0][j], p2 = (j == 1 ? 1.0 : 0.0) + 0.5 * M[1][j];
#pragma unroll
          for (int i = 0; i < 2; ++i)
            M[i][j] = g.dt * (vx[i][0] * p1 + vx[i][1] * p2 + (j >= 2 ? vu[i][j >= 2 ? j - 2 : 0] : 0.0));
        }
        d1 = g.dt * v[0];
        d2 = g.dt * v[1];
      }
      const double y1b = x1b, y2b = x2b;
      x1b += M[0][0] * y1b + M[1][0] * y2b;
      x2b += M[0][1] * y1b + M[1][1] * y2b;
      u1b += M[0][2] * y1b + M[1][2] * y2b;
      u2b += M[0][3] * y1b + M[1][3] * y2b;
      u3b += M[0][4] * y1b + M[1][4] * y2b;
    }
  }

  FrameBar m = {};
  double Eb[3] = {0.0, 0.0, 0.0}, Bb[3] = {0.0, 0.0, 0.0};
  if (qm != 0.0) em_reverse(f, E, B, kb, z1, z2, a3, u1b, u2b, u3b, Eb, Bb, m);

  // momentum stage, backwards
  if (fixed_u) {
    const double b1 = 0.5 * (a1 + z1), b2 = 0.5 * (a2 + z2), hd = 0.5 * g.dt;
    double fb[2][2];
    force_jac<kMap>(g, f, d, e, b1, b2, fb);
    const double c11 = 1.0 - hd * fb[0][0], c22 = 1.0 - hd * fb[1][1], c12 = hd * fb[1][0], c21 = hd * fb[0][1];
    const double id = 1.0 / (c11 * c22 - c12 * c21);
    const double l1 = (c22 * u1b + c12 * u2b) * id, l2 = (c21 * u1b + c11 * u2b) * id;
    double b1b, b2b;
    force_reverse<kMap>(g, f, d, e, a3, b1, b2, g.dt * l1, g.dt * l2, b1b, b2b, u3b, m);
    u1b = l1 + 0.5 * b1b;
    u2b = l2 + 0.5 * b2b;
  } else {
    // through the n_iter iterations run, last to first
    double z1b = u1b, z2b = u2b;
    u1b = u2b = 0.0;
    reverse_iterates<16>(
        g.n_iter, a1, a2, [&](double& y1, double& y2) { momentum_map<kMap>(g, f, d, e, y1, y2, y1, y2); },
        [&](double y1, double y2) {
          double b1b, b2b;
          force_reverse<kMap>(g, f, d, e, a3, 0.5 * (a1 + y1), 0.5 * (a2 + y2), g.dt * z1b, g.dt * z2b, b1b, b2b, u3b, m);
          u1b += z1b + 0.5 * b1b;
          u2b += z2b + 0.5 * b2b;
          z1b = 0.5 * b1b;
          z2b = 0.5 * b2b;
        });
    u1b += z1b;  // the first iterate starts from Z = s
    u2b += z2b;
  }

  if (qm != 0.0) {
    em_reverse(f, E, B, kb, st.u1, st.u2, st.u3, u1b, u2b, u3b, Eb, Bb, m);
    double F[6], Fb[6];
    gather(g, fp, i1, dx1, i2, dx2, F);
    tetrad_reverse(f, F, Eb, Fb, m);
    tetrad_reverse(f, F + 3, Bb, Fb + 3, m);
    double fsum = 0.0;
    gather_reverse(g, fp, i1, dx1, i2, dx2, Fb, x1b, x2b, fsum);
    gB0 += fsum * inv_B0;
  }
  // the metric's bars back to the position
  FrameT<T2> ft;
  GradT<T2> dt2;
  frame_from<kMap>(g, rsc_tan(g, p, x2), &ft, &dt2);
  double xb[2] = {x1b, x2b};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    xb[j] += m.alpha * ft.c.alpha.d[j] + m.hu11 * ft.c.hu11.d[j] + m.hu13 * ft.c.hu13.d[j] + m.hu22 * ft.c.hu22.d[j] +
             m.hu33 * ft.c.hu33.d[j] + m.is11 * ft.is11.d[j] + m.s22 * ft.s22.d[j] + m.s33 * ft.s33.d[j] +
             m.is33 * ft.is33.d[j];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      xb[j] += m.da[i] * dt2.alpha[i].d[j] + m.db[i] * dt2.beta1[i].d[j] + m.l11[i] * dt2.l11[i].d[j] +
               m.z[i] * dt2.z[i].d[j];
    xb[j] += m.ct * dt2.ct.d[j];
    if (kMap) xb[j] += m.tt * dt2.tt.d[j];
  }
  gbar[0] = xb[0];
  gbar[1] = xb[1];
  gbar[2] = u1b;
  gbar[3] = u2b;
  gbar[4] = u3b;
}

// gin, gout: 5 x n (SoA rows x1, x2, u1, u2, u3); may alias.  gB0: n, accumulated.
constexpr int kAdjBlock = 64;
template <int SER>
__global__ void __launch_bounds__(kAdjBlock) push_adjoint_kernel(Grid g, Tables tab, GatherPlanesT<double> fp,
                                                                 double inv_B0, ParticleArrays P, const double* gin,
                                                                 double* gout, double* gB0) {
  const int64_t k0 = (int64_t)blockIdx.x * kAdjBlock, k = k0 + threadIdx.x;
  if (k >= P.n) return;
  double a[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) a[c] = gin[c * P.n + k];
  double acc = gB0[k];
  adjoint_one<SER>(g, tab, fp, inv_B0, from_slot(P, k0), threadIdx.x, a, acc);
#pragma unroll
  for (int c = 0; c < 5; ++c) gout[c * P.n + k] = a[c];
  gB0[k] = acc;
}

}  // namespace grpic
