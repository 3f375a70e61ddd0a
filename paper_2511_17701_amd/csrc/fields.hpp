// fields.hpp -- field-solver kernels (Sec. 3.3, 3.4).
//
// Kernels are templated on the storage type T of the planes (double, or float
// in the single-precision form); the metric weights and the update arithmetic
// are FP64 and each result is rounded once on store.
//
// Threads run along theta (the contiguous index of a plane), blocks along r.
// Geometry at staggered grid points is assembled from 1-D tables of r and
// 1/(R deta) at integer / half-integer x1 and of sin, cos, 1/sin (and, when
// h0 != 0, T = dtheta/dx2 and deta/T) at integer / half-integer x2, with one
// reciprocal square root per point; R = dr/dx1 = dxi (r - r0).
#pragma once

#include "geometry.hpp"

namespace grpic {

__device__ inline Cell cell_tab(const Grid& g, const Tables& t, int i, int o1, int j, int o2) {
  const double r = t.r[o1][i + g.ng], R = g.dxi * (r - g.r0);
  const double s = t.s[o2][j + g.ng], c = t.c[o2][j + g.ng];
  const double T = g.h0 == 0.0 ? g.dth : t.td[o2][j + g.ng];
  const double a2 = g.a * g.a, r2 = r * r, tMr = 2.0 * g.M * r;
  const double Sig = r2 + a2 * c * c;
  const double S2 = Sig + tMr;
  const double ra = r2 + a2;
  const double A = ra * ra - a2 * (ra - tMr) * s * s;
  const double opz = S2 / Sig;
  Cell e;
  e.alpha = sqrt(Sig / S2);
  e.beta1 = tMr / (S2 * R);
  e.hl11 = opz * R * R;
  e.hl22 = Sig * T * T;
  e.hl33 = A * s * s / Sig;
  e.hl13 = -g.a * opz * s * s * R;
  e.sqrt_ht = R * T * Sig / e.alpha;
  e.sqrt_h = e.sqrt_ht * s;
  return e;
}

// ---------------------------------------------------------------- weights
// Solver weights at one staggered point (i + o1/2, j + o2/2).  With
// S2 = Sigma + 2 M r and k = 1/sqrt(Sigma S2), the lapse is Sigma k,
// 1/Sigma = S2 k^2, 1/S2 = Sigma k^2 and sqrt(h)/sin(theta) = R T / k
// (R = dr/dx1, T = dtheta/dx2), so one reciprocal square root gives every factor of the
// closed forms of App. A (the same quantities as cell_tab).
struct FW {
  double alpha;                   // lapse
  double hl11, hl22, hl33;        // lower spatial metric, code components
  double w13;                     // sqrt(h)/sin * h_13       (radial-average weight)
  double wb;                      // sqrt(h)/sin * sqrt(h) * beta^1
  double h_sht;                   // 1 / (2 sqrt(h)/sin)      (radial-average norm)
  double ish;                     // 1 / sqrt(h)              (0 on the axis)
};

// kQ: the general quasi-spherical map (r0, h0 not both 0); otherwise the
// logarithmic-r, uniform-theta grid, with R = dxi r and T = deta.
template <bool kQ>
__device__ inline FW fw_tab(const Grid& g, const Tables& t, int i, int o1, int j, int o2) {
  const uint32_t ic = (uint32_t)(i + g.ng), jc = (uint32_t)(j + g.ng);
  const double r = t.r[o1][ic], R = g.dxi * (kQ ? r - g.r0 : r);
  const double s = elem(t.s[o2], jc), c = elem(t.c[o2], jc), is = elem(t.is[o2], jc);
  const double T = kQ ? elem(t.td[o2], jc) : g.dth;
  const double ird = kQ ? t.ird[o1][ic] * elem(t.eta_t[o2], jc) : t.ird[o1][ic];  // 1/(R T)
  const double a2 = g.a * g.a, r2 = r * r, tMr = 2.0 * g.M * r, s2 = s * s;
  const double Sig = r2 + a2 * c * c;
  const double S2 = Sig + tMr;
  const double ra = r2 + a2;
  const double A = ra * ra - a2 * (ra - tMr) * s2;
  const double k = rsqrt(Sig * S2);
  const double k2 = k * k;
  const double S2k = S2 * k;
  FW e;
  e.alpha = Sig * k;
  e.hl11 = S2k * S2k * R * R;
  e.hl22 = Sig * T * T;
  e.hl33 = A * s2 * S2 * k2;
  e.w13 = -g.a * T * R * R * s2 * S2 * S2k;
  e.wb = R * T * T * s * tMr * Sig;
  e.h_sht = 0.5 * k * ird;
  e.ish = k * ird * is;
  return e;
}

template <class T>
struct TriT {
  T* __restrict__ p[3];
};
template <class T>
struct CTriT {
  const T* __restrict__ p[3];
};
using Tri = TriT<double>;
using CTri = CTriT<double>;

// The launch's row of a field-stage thread.  A block is 2 rows of 128 threads,
// so a wavefront lies in one row: the row is made a scalar, with it the r
// tables' values and the plane rows' addresses (pt).
__device__ inline int launch_row() {
  return __builtin_amdgcn_readfirstlane((int)(blockIdx.y * blockDim.y + threadIdx.y));
}
__device__ inline int launch_col() { return (int)(blockIdx.x * blockDim.x + threadIdx.x); }

// Plane point (i, j): a scalar row base and a 32-bit column offset.
template <class T>
__device__ inline T& pt(const Grid& g, T* __restrict__ p, int i, int j) {
  return elem(p + (int64_t)(i + g.ng) * g.ld, (uint32_t)(j + g.ng));
}

// Plane point (i, j) of a if first, else of b.
template <class T>
__device__ inline T pt_of(const Grid& g, bool first, const T* __restrict__ a, const T* __restrict__ b, int i, int j) {
  return (first ? a : b)[(int64_t)(i + g.ng) * g.ld + (j + g.ng)];
}

// ---------------------------------------------------------------- aux E, H
// eq. discretized-auxE/-auxH with the volume-weighted radial averages of
// Sec. 3.3.1 (weights sqrt(h)/sin(theta)); for i in [-1, n_r], j in [0, n_th].
// kE / kH select the outputs; both read the same B, D and share the weights.
template <class T, bool kE, bool kH, bool kQ>
__global__ void aux_kernel(Grid g, Tables t, CTriT<T> Bs, CTriT<T> Ds, TriT<T> E, TriT<T> H) {
  const int j = launch_col(), i = launch_row() - 1;
  if (j > g.n_th || i > g.n_r) return;
  const bool half = j < g.n_th;  // theta-staggered components exist
  // weights at the points the stencils touch (unused ones are not computed)
  const FW n00 = fw_tab<kQ>(g, t, i, 0, j, 0);       // (i, j)
  const FW n10 = fw_tab<kQ>(g, t, i + 1, 0, j, 0);   // (i+1, j)
  const FW h00 = fw_tab<kQ>(g, t, i, 1, j, 0);       // (i+1/2, j)
  const FW hm0 = fw_tab<kQ>(g, t, i - 1, 1, j, 0);   // (i-1/2, j)
  const FW n01 = fw_tab<kQ>(g, t, i, 0, j, 1);       // (i, j+1/2)
  const FW n11 = fw_tab<kQ>(g, t, i + 1, 0, j, 1);   // (i+1, j+1/2)
  const FW h01 = fw_tab<kQ>(g, t, i, 1, j, 1);       // (i+1/2, j+1/2)
  const FW hm1 = fw_tab<kQ>(g, t, i - 1, 1, j, 1);   // (i-1/2, j+1/2)
  if (kE) {
    {  // E_1 (i+1/2, j)
      const double av = (n00.w13 * pt(g, Ds.p[2], i, j) + n10.w13 * pt(g, Ds.p[2], i + 1, j)) * h00.h_sht;
      pt(g, E.p[0], i, j) = h00.alpha * (h00.hl11 * pt(g, Ds.p[0], i, j) + av);
    }
    {  // E_3 (i, j)
      const double a1 = (hm0.w13 * pt(g, Ds.p[0], i - 1, j) + h00.w13 * pt(g, Ds.p[0], i, j)) * n00.h_sht;
      const double a2 = (hm0.wb * pt(g, Bs.p[1], i - 1, j) + h00.wb * pt(g, Bs.p[1], i, j)) * n00.h_sht;
      pt(g, E.p[2], i, j) = n00.alpha * (n00.hl33 * pt(g, Ds.p[2], i, j) + a1) + a2;
    }
    if (half) {  // E_2 (i, j+1/2)
      const double a3 = (hm1.wb * pt(g, Bs.p[2], i - 1, j) + h01.wb * pt(g, Bs.p[2], i, j)) * n01.h_sht;
      pt(g, E.p[1], i, j) = n01.alpha * n01.hl22 * pt(g, Ds.p[1], i, j) - a3;
    }
  }
  if (kH) {
    {  // H_2 (i+1/2, j)
      const double a1 = (n00.wb * pt(g, Ds.p[2], i, j) + n10.wb * pt(g, Ds.p[2], i + 1, j)) * h00.h_sht;
      pt(g, H.p[1], i, j) = h00.alpha * h00.hl22 * pt(g, Bs.p[1], i, j) + a1;
    }
    if (half) {
      {  // H_1 (i, j+1/2)
        const double a2 = (hm1.w13 * pt(g, Bs.p[2], i - 1, j) + h01.w13 * pt(g, Bs.p[2], i, j)) * n01.h_sht;
        pt(g, H.p[0], i, j) = n01.alpha * (n01.hl11 * pt(g, Bs.p[0], i, j) + a2);
      }
      {  // H_3 (i+1/2, j+1/2)
        const double a3 = (n01.w13 * pt(g, Bs.p[0], i, j) + n11.w13 * pt(g, Bs.p[0], i + 1, j)) * h01.h_sht;
        const double a4 = (n01.wb * pt(g, Ds.p[1], i, j) + n11.wb * pt(g, Ds.p[1], i + 1, j)) * h01.h_sht;
        pt(g, H.p[2], i, j) = h01.alpha * (h01.hl33 * pt(g, Bs.p[2], i, j) + a3) - a4;
      }
    }
  }
}

// ---------------------------------------------------------------- boundaries
// An updated triple X and what its boundary conditions need:
//  - constant layer inside the horizon: rows i <= n_f take row n_f + 1;
//  - absorbing layer: F <- F - lambda (F - F_init), lambda a cubic ramp over
//    the last n_absorb cells (and beyond);
//  - axis reflection (Sec. 3.3.3): r-components even, theta and phi
//    components odd; the component `zero` (B^2, D^3) vanishes on the axis rows.
// L: in the single-precision form the evolved fields D and B carry a
// compensation plane (null otherwise): X + L holds the running sum to about 48
// bits and X, what every reader sees, is its rounding to float, so rounding
// errors of the time integration do not accumulate step after step.
// S: receives X as it was before the update, ghosts included (null: not kept).
template <class T>
struct UpdateT {
  TriT<T> X, L;
  CTriT<T> X0;  // targets of the absorbing layer
  TriT<T> S;
  int3 half1, half2;  // staggering of the components in x1, x2
  int zero;
  int edge;  // the row from which the update writes the horizon rows: n_f + 1, or
             // none (-1: horizon_kernel follows)
};

// Where the threads of row n_f + 1 write the horizon rows of their column, one
// after the other: for few rows, and for some more where the rest of the update
// is long enough to hide them.  Elsewhere a launch more (horizon_kernel) is
// shorter.  A step's field stages with the rows in the updates / in launches of
// their own, us: 64^2 in double precision n_f = 4 65.3 / 64.2, 6 78.7 / 74.0, 8
// 88.5 / 80.2, 24 177 / 130; 512^2 4 96.3 / 98.3, 6 114 / 109, 24 230 / 177;
// 2048^2 4 825 / 837, 8 866 / 878, 16 958 / 963, 24 1066 / 1054 (single
// precision: the same order, 8 at 512^2 115 / 108, at 2048^2 614 / 625).
__host__ __device__ inline bool horizon_in_update(const Grid& g) {
  return g.n_filter <= 4 || (g.n_filter <= 16 && g.plane >= (int64_t)1 << 21);
}

// Stores v, the updated component c at (i, j), i > n_f, j an interior column of
// the component, through the boundary conditions.  The thread that owns the
// point also writes the ghost columns that mirror it and, from row u.edge, the
// horizon rows (and saves what was there): every stored value has one writer
// and no reader among the other threads, so an update and its boundaries are one
// pass.  was: the stored value before (the update's kernels load everything
// before their first store).  As passes of their own (two launches per updated triple, eight per
// step) they took 38 us of a 354 us step at 512^2 and 24 of 79 at 40 x 56.
// Five steps of the field stages at 1537 x 1023 in double precision: 1912 ->
// 1707 us, of which the scalar rows give 40 and the loads ahead of the stores 100.
template <class T>
__device__ inline void store_bc(const Grid& g, const UpdateT<T>& u, int c, int i, int j, double v, T was) {
  T* const X = u.X.p[c];
  T* const S = u.S.p[0] ? u.S.p[c] : nullptr;
  const bool comp = sizeof(T) == 4 && u.L.p[0];
  const int h1 = c == 0 ? u.half1.x : c == 1 ? u.half1.y : u.half1.z;
  const int h2 = c == 0 ? u.half2.x : c == 1 ? u.half2.y : u.half2.z;
  const int n = g.n_th;
  if (g.n_absorb > 0) {
    const double x = (double)i + 0.5 * h1, x0 = (double)(g.n_r - g.n_absorb);
    if (x > x0) {
      const double sr = fmin((x - x0) / g.n_absorb, 1.0);
      const double lam = sr * sr * sr;
      v = v - lam * (v - (double)pt(g, u.X0.p[c], i, j));
    }
  }
  if (c == u.zero && (j == 0 || j == n)) v = 0.0;
  const T h = (T)v, l = (T)(v - (double)h);
  if (S) pt(g, S, i, j) = was;
  pt(g, X, i, j) = h;
  if (comp) pt(g, u.L.p[c], i, j) = l;
  // column q of the rows [first, last], a few at a time (their loads together)
  auto put = [&](int first, int last, int q, T w) {
    constexpr int kRows = 4;
    for (int r0 = first; r0 <= last; r0 += kRows) {
      T old[kRows];
      if (S) {
#pragma unroll
        for (int e = 0; e < kRows; ++e)
          if (r0 + e <= last) old[e] = pt(g, X, r0 + e, q);
      }
#pragma unroll
      for (int e = 0; e < kRows; ++e)
        if (r0 + e <= last) {
          if (S) pt(g, S, r0 + e, q) = old[e];
          pt(g, X, r0 + e, q) = w;
        }
    }
  };
  const bool edge = i == u.edge;
  if (edge) {
    put(-g.ng, i - 1, j, h);
    if (comp)
      for (int r = -g.ng; r < i; ++r) pt(g, u.L.p[c], r, j) = l;
  }
  // the ghost column that mirrors column j
  const int lo = h2 ? j : j - 1;  // 0: column -1, 1: column -2
  const int hi = n - 1 - j;       // half: 0: column n, 1: column n + 1; node: 0: column n + 1
  const bool low = lo == 0 || lo == 1, high = h2 ? hi == 0 || hi == 1 : hi == 0;
  if (low | high) put(edge ? -g.ng : i, i, low ? -1 - lo : h2 ? n + hi : n + 1, c == 0 ? h : -h);
}

// The horizon rows of an updated triple as a pass of its own, one thread per
// point of the rows [-ng, n_f]: what was there goes to S, the value (and
// compensation) of row n_f + 1 takes its place.  For many filter passes, where
// store_bc's walk over the rows would outlast the rest of the update.
template <class T>
__global__ void horizon_kernel(Grid g, UpdateT<T> u) {
  const int j = launch_col() - g.ng, i = launch_row() - g.ng, e = g.n_filter + 1;
  if (j >= g.n_th + g.ng || i >= e) return;
  T was[3], h[3], l[3];
  const bool comp = sizeof(T) == 4 && u.L.p[0];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    was[c] = pt(g, u.X.p[c], i, j);
    h[c] = pt(g, u.X.p[c], e, j);
    l[c] = comp ? pt(g, u.L.p[c], e, j) : (T)0;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (u.S.p[0]) pt(g, u.S.p[c], i, j) = was[c];
    pt(g, u.X.p[c], i, j) = h[c];
    if (comp) pt(g, u.L.p[c], i, j) = l[c];
  }
}

// ---------------------------------------------------------------- Faraday
// eq. discretized-faraday on the evolved ranges i in [0, n_r], j in [0, n_th],
// and the boundaries of the updated triple; one thread per point of the rows
// n_f < i < n_r + ng and the columns [0, n_th].  kPre: the triple is averaged
// with A first, X <- (X + A)/2 + update (Sec. 3.4, step 2).
template <class T, bool kPre, bool kQ>
__global__ void faraday_kernel(Grid g, Tables t, UpdateT<T> u, CTriT<T> E, CTriT<T> A) {
  const int j = launch_col(), i = launch_row() + g.n_filter + 1;
  if (j > g.n_th || i >= g.n_r + g.ng) return;
  const bool half = j < g.n_th;  // theta-staggered components exist
  // (in column n_th they are ghosts, which the threads of column n_th - 1 write)
  T was[3] = {}, add[3] = {};  // the stored values and what is added to them: A or the compensation
  auto load = [&](int c) {
    was[c] = pt(g, u.X.p[c], i, j);
    if (kPre) add[c] = pt(g, A.p[c], i, j);
    else if (sizeof(T) == 4 && u.L.p[0]) add[c] = pt(g, u.L.p[c], i, j);
  };
  load(1);
  if (half) {
    load(0);
    load(2);
  }
  double v[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) v[c] = (kPre ? 0.5 : 1.0) * ((double)was[c] + (double)add[c]);
  if (i <= g.n_r) {
    const bool below = i < g.n_r;
    const double e3 = (double)pt(g, E.p[2], i, j);
    if (half) v[0] -= g.dt * ((double)pt(g, E.p[2], i, j + 1) - e3) * fw_tab<kQ>(g, t, i, 0, j, 1).ish;
    if (below && j >= 1 && half) v[1] += g.dt * ((double)pt(g, E.p[2], i + 1, j) - e3) * fw_tab<kQ>(g, t, i, 1, j, 0).ish;
    if (below && half) {
      const double curl = ((double)pt(g, E.p[1], i + 1, j) - (double)pt(g, E.p[1], i, j)) -
                          ((double)pt(g, E.p[0], i, j + 1) - (double)pt(g, E.p[0], i, j));
      v[2] -= g.dt * curl * fw_tab<kQ>(g, t, i, 1, j, 1).ish;
    }
  }
  if (half) store_bc(g, u, 0, i, j, v[0], was[0]);
  store_bc(g, u, 1, i, j, v[1], was[1]);
  if (half) store_bc(g, u, 2, i, j, v[2], was[2]);
}

// ---------------------------------------------------------------- Ampere
// eq. discretized-ampere with the current J = wa Ja + wb Jb, and the boundaries
// of the updated triple; D^1 on the axis rows from the polar-cap integral form
// (Sec. 3.3.2): cap area A_{i+1/2}, the printed 2 pi with the two-sided
// (mirrored) axis-row current the deposit leaves there; the theta = pi cap has
// the opposite orientation.  kFinal (the last half of the step): the grid spans
// the whole plane, the current is Ja alone, and the same pass rotates the
// currents: Jb <- Ja, and the deposit's accumulator is zeroed (Jclear, or Ja
// itself when Jclear is null: the filter leaves the filtered current in the
// scratch set or in the accumulator).
template <class T, bool kFinal, bool kQ>
__global__ void ampere_kernel(Grid g, Tables t, UpdateT<T> u, CTriT<T> H, TriT<T> Ja, TriT<T> Jb, double wa, double wb,
                              double polar_k, TriT<T> Jclear) {
  const int j = launch_col() - (kFinal ? g.ng : 0), i = launch_row() + (kFinal ? -g.ng : g.n_filter + 1);
  if (j >= g.n_th + g.ng || i >= g.n_r + g.ng) return;
  T ja[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) ja[c] = pt(g, Ja.p[c], i, j);
  if (i > g.n_filter && j >= 0 && j <= g.n_th) {
    const bool half = j < g.n_th;  // theta-staggered components exist
    T was[3];
    double v[3], J[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      // component 1 in column n_th is a ghost, which the thread of column n_th - 1
      // writes: a value of its target plane instead (unused), since a branch
      // around these loads costs 6 % of the pass (4096^2, single precision)
      const bool own = half || c != 1;
      was[c] = pt_of(g, own, u.X.p[c], u.X0.p[c], i, j);
      const double add = sizeof(T) == 4 && u.L.p[0] ? (double)pt_of(g, own, u.L.p[c], u.X0.p[c], i, j) : 0.0;
      v[c] = (double)was[c] + add;
      J[c] = kFinal ? (double)ja[c] : wa * (double)ja[c] + wb * (double)pt(g, Jb.p[c], i, j);
    }
    const double fpi = 4.0 * kPi;
    if (i <= g.n_r) {
      const double h3 = (double)pt(g, H.p[2], i, j);
      if (i < g.n_r) {
        const double h3m = (double)pt(g, H.p[2], i, j - 1);
        if (j >= 1 && half) {
          v[0] += g.dt * ((h3 - h3m) - fpi * J[0]) * fw_tab<kQ>(g, t, i, 1, j, 0).ish;
        } else {
          const double r = t.r[1][i + g.ng];
          const double ra = r * r + g.a * g.a;
          const double Ap = g.dxi * (kQ ? r - g.r0 : r) * ra * sqrt(1.0 + 2.0 * g.M * r / ra) * polar_k;
          v[0] += g.dt * ((j == 0 ? h3 : -h3m) - 2.0 * kPi * J[0]) / Ap;
        }
      }
      if (half) v[1] += g.dt * (-(h3 - (double)pt(g, H.p[2], i - 1, j)) - fpi * J[1]) * fw_tab<kQ>(g, t, i, 0, j, 1).ish;
      if (j >= 1 && half) {
        const double curl = ((double)pt(g, H.p[1], i, j) - (double)pt(g, H.p[1], i - 1, j)) -
                            ((double)pt(g, H.p[0], i, j) - (double)pt(g, H.p[0], i, j - 1));
        v[2] += g.dt * (curl - fpi * J[2]) * fw_tab<kQ>(g, t, i, 0, j, 0).ish;
      }
    }
    store_bc(g, u, 0, i, j, v[0], was[0]);
    if (half) store_bc(g, u, 1, i, j, v[1], was[1]);
    store_bc(g, u, 2, i, j, v[2], was[2]);
  }
  if (kFinal) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      pt(g, Jb.p[c], i, j) = ja[c];
      pt(g, Jclear.p[0] ? Jclear.p[c] : Ja.p[c], i, j) = 0.0;
    }
  }
}

// ---------------------------------------------------------------- axis reflection of initial data
// 6 ng lanes per plane row, one per (component, ghost column): bc_axis_rows
// rows per block of `threads`.
__host__ __device__ inline int bc_axis_rows(const Grid& g, int threads) { return threads / (6 * g.ng); }

// Axis reflection of every plane row: each ghost column of a component is
// the reflection of its mirror column (node rows run 0..n, half rows
// 0..n-1); the mirrors are interior columns, which this pass only zeroes at
// j = 0, n for zero_comp, and never reads.
template <class T>
__global__ void bc_axis_kernel(Grid g, TriT<T> X, int3 half2, int zero_comp) {
  const int lanes = 6 * g.ng, rpb = bc_axis_rows(g, (int)blockDim.x);
  const int t = (int)threadIdx.x;
  const int i = (int)blockIdx.x * rpb + t / lanes - g.ng;
  if (t >= rpb * lanes || i >= g.n_r + g.ng) return;
  const int h2[3] = {half2.x, half2.y, half2.z};
  const int c = (t % lanes) / (2 * g.ng), q = (t % lanes) % (2 * g.ng);
  const int n = g.n_th;
  T* C = X.p[c];
  const int j = q < g.ng ? -1 - q : n - h2[c] + 1 + (q - g.ng);  // ghost column
  const bool exists = j < n + g.ng;
  const int m = j < 0 ? (h2[c] ? -1 - j : -j) : (h2[c] ? 2 * n - 1 - j : 2 * n - j);
  const T v = exists ? C[ix(g, i, m)] : (T)0;
  if (exists) C[ix(g, i, j)] = (c == 0 ? 1.0 : -1.0) * v;
  if (!h2[c] && c == zero_comp && (q == 0 || q == g.ng)) {
    const int jz = q == 0 ? 0 : n;
    C[ix(g, i, jz)] = 0.0;
  }
}

// ---------------------------------------------------------------- misc
// elementwise over whole planes (ghosts included)
template <class T>
__global__ void average_kernel(int64_t n, TriT<T> A, CTriT<T> B) {  // A <- (A + B) / 2
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) A.p[c][k] = 0.5 * (A.p[c][k] + B.p[c][k]);
}

// Initial data are launch-bound on the grids of frozen-field runs, which build
// them for every amplitude: a field set is cleared in one launch and copied in
// one (33 and 4 before: 85 of the 270 us that five steps of 1e3 particles
// kept the GPU busy with, forward and back).
constexpr int kMaxPlanes = 39;
template <class T>
struct PlaneSetT {
  T* p[kMaxPlanes];
};
template <class T>
__global__ void clear_planes_kernel(int64_t n, PlaneSetT<T> s) {  // plane blockIdx.y
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) s.p[blockIdx.y][k] = (T)0;
}

template <class T>
__global__ void copy_initial_kernel(int64_t n, CTriT<T> D, CTriT<T> B, TriT<T> D0, TriT<T> B0, TriT<T> Di, TriT<T> Bi) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    D0.p[c][k] = Di.p[c][k] = D.p[c][k];
    B0.p[c][k] = Bi.p[c][k] = B.p[c][k];
  }
}

template <class T>
__global__ void fill_kernel(int64_t n, T* __restrict__ p, double v) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = v;
}

// ---------------------------------------------------------------- filter
// Binomial passes (1,2,1)/4 x (1,2,1)/4 of a current plane (Sec. 3.3.4), in
// the arithmetic of one pass at plane point (i, j) of a component of
// x2-staggering hs and axis parity par, reading the source S of the pass:
//  - ghost columns (j < 0 or j > n_th - hs) take the source's axis reflection
//    par S(i, mirror(j));
//  - the two outermost plane rows keep the source;
//  - every other point is (R(i-1) + 2 R(i) + R(i+1)) / 16 rounded to T, with
//    the FP64 row sums R(i) = pm S(i, j-1) + 2 S(i, j) + pp S(i, j+1), whose
//    theta neighbours past an axis are read as reflections (pm, pp = par
//    there, 1 elsewhere).
// Every product is by 1, 2 or a power of two, so the result does not depend
// on how the compiler contracts the sums.
//
// Up to kFMaxPasses passes run in one launch.  A wavefront owns a strip of
// 64 plane columns (one per lane) and kSR output rows, and holds its rows plus
// a halo of P rows on each side in registers for the whole run: the theta
// neighbours come from the adjacent lanes by DPP wave shifts and the axis
// reflections by a lane permute (only in strips that touch an axis); the
// radial sums slide down the rows.  No LDS and no barriers.  Values whose
// neighbours lie outside the strip (the wave's first and last lane, the first
// and last staged row) are not computed: the stale points move inwards by one
// per pass, so after P passes the 56 middle lanes and the kSR middle rows are
// exact; at the plane's edges nothing outside is needed and the strip outputs
// up to the edge.  The last strip of a row is shifted to end at the plane's
// last column, so the far-axis reflections it reads are exact (the columns it
// shares with its neighbour get identical values twice).  X must not alias S.
constexpr int kFMaxPasses = 4;
constexpr int kFLanes = 64, kFOut = kFLanes - 2 * kFMaxPasses;  // 56 output columns per strip

// number of 64-column strips that cover a plane row of ld stored columns,
// and the first stored column of strip b (the last one ends at the plane's
// last column)
__host__ __device__ inline int filter_strips_theta(int ld) {
  return ld <= kFLanes ? 1 : (ld - (kFLanes - kFMaxPasses) + kFOut - 1) / kFOut + 1;
}
__host__ __device__ inline int filter_strip_lo(int b, int ld) {
  return min(b * kFOut, max(ld - kFLanes, 0));
}
// whether strip b touches an axis (a column j <= 0 or j >= n_th - 1)
__host__ __device__ inline bool filter_strip_axis(int b, int ld, int n, int ng) {
  const int lo = filter_strip_lo(b, ld);
  return lo <= ng || lo + kFLanes - 1 >= n - 1 + ng;
}

// the lane's value one lane down (wave_shr:1) and one lane up (wave_shl:1);
// the first / last lane reads 0
__device__ inline int lane_down(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, false); }
__device__ inline int lane_up(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, false); }
__device__ inline float lane_down(float v) { return __int_as_float(lane_down(__float_as_int(v))); }
__device__ inline float lane_up(float v) { return __int_as_float(lane_up(__float_as_int(v))); }
__device__ inline double lane_down(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_down((int)(b & 0xffffffffll)), hi = lane_down((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}
__device__ inline double lane_up(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_up((int)(b & 0xffffffffll)), hi = lane_up((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

// Column j reflected across the axis for a component of x2-staggering hs
// (node rows run 0..n, half rows 0..n-1); interior columns map to themselves.
__device__ inline int axis_mirror(int j, int n, int hs) {
  if (j < 0) return hs ? -1 - j : -j;
  if (j > n - hs) return hs ? 2 * n - 1 - j : 2 * n - j;
  return j;
}

// Lane-constant data of one component in a strip that touches an axis.
struct FilterAxis {
  bool lo, hi;     // j == 0 / j == n - hs: the theta neighbour past the axis is a reflection
  bool ghost;      // ghost column
  int src;         // lane of the reflected column (ghost lanes)
  bool hs;         // half-staggered in x2
  double par;      // axis parity
};

// FP64 theta row sum of the pass at this lane
template <class T, bool kAxis>
__device__ inline double filter_row_sum(T a, const FilterAxis& ax) {
  const T dn = lane_down(a), up = lane_up(a);
  double lv = (double)dn, rv = (double)up;
  if (kAxis) {
    if (ax.lo) lv = ax.par * (double)(ax.hs ? a : up);
    if (ax.hi) rv = ax.par * (double)(ax.hs ? a : dn);
  }
  return (lv + 2.0 * (double)a) + rv;
}

// One component of a strip: load, P passes, store rows [rlo, rhi).  kAxis:
// the strip touches an axis (reflected neighbours, ghost columns); kRows: a
// plane of fewer rows than a strip stages (rows outside the plane, the two
// kept rows inside the strip).  Otherwise the strips are placed so that the
// kept rows are a strip's first or last staged row, which no pass updates.
template <class T, int P, int kSR, bool kAxis, bool kRows>
__device__ __forceinline__ void filter_strip_comp(const Grid& g, T* __restrict__ x, const T* __restrict__ s,
                                                  int J, bool col, bool out, int ifirst, int rlo, int rhi,
                                                  const FilterAxis& ax) {
  constexpr int R = kSR + 2 * P;
  // one wavefront-uniform base (the strip's first staged row) and 32-bit
  // per-lane byte offsets (a strip spans R rows: far below 4 GiB)
  const int64_t row0 = (int64_t)(ifirst + g.ng) * g.ld;
  const char* __restrict__ sb = (const char*)(s + row0);
  const uint32_t rowb = (uint32_t)(g.ld * sizeof(T)), lb = (uint32_t)(J * sizeof(T));
  T v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = ifirst + r;
    v[r] = col && (!kRows || (i >= -g.ng && i < g.n_r + g.ng)) ? *(const T*)(sb + (lb + (uint32_t)r * rowb))
                                                                : (T)0;
    if ((r & 7) == 7) __builtin_amdgcn_sched_barrier(0);  // 8 row offsets live at a time
  }
#pragma unroll 1
  for (int p = 0; p < P; ++p) {
    double s_prev = 0.0, s_cur = filter_row_sum<T, kAxis>(v[0], ax);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double s_next = r + 1 < R ? filter_row_sum<T, kAxis>(v[r + 1], ax) : 0.0;
      const int i = ifirst + r;
      T nv = v[r];
      if (r >= 1 && r <= R - 2 && (!kRows || (i >= 1 - g.ng && i <= g.n_r + g.ng - 2)))
        nv = (T)(0.0625 * ((s_prev + 2.0 * s_cur) + s_next));
      if (kAxis) {
        const T m = __shfl(v[r], ax.src);
        if (ax.ghost) nv = (T)(ax.par * (double)m);
      }
      v[r] = nv;
      s_prev = s_cur;
      s_cur = s_next;
      __builtin_amdgcn_sched_barrier(0);  // row by row: a few sums live, not all
    }
  }
  if (out) {
    // an opaque copy of the lane offset: the stores recompute their row
    // offsets instead of keeping the loads' live through the passes
    uint32_t lbs = lb;
    asm volatile("" : "+v"(lbs));
    char* __restrict__ db = (char*)(x + row0);
    auto put = [&](int r) { *(T*)(db + (lbs + (uint32_t)r * rowb)) = v[r]; };
    if (kRows) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r >= rlo && r < rhi && ifirst + r < g.n_r + g.ng) put(r);
    } else {  // rows [rlo, rhi) = [P or 0, P + kSR or R)
#pragma unroll
      for (int r = P; r < P + kSR; ++r) put(r);
      if (rlo == 0) {
#pragma unroll
        for (int r = 0; r < P; ++r) put(r);
      }
      if (rhi == R) {
#pragma unroll
        for (int r = P + kSR; r < R; ++r) put(r);
      }
    }
  }
}

// number of row strips of a plane with nrow rows (kRows: nrow < kSR + 2 P)
template <int P, int kSR, bool kRows>
__host__ __device__ inline int filter_strips_r(int nrow) {
  return kRows ? (nrow + kSR - 1) / kSR : (nrow - (kSR + 2 * P) + kSR - 1) / kSR + 1;
}

// P passes of S into X, plane blockIdx.z.  Grid: (filter_strips_theta(ld),
// ceil(filter_strips_r / 4), number of planes); 256 threads = 4 wavefronts on
// consecutive row strips.  Strip s stages rows from min(s kSR - ng,
// n_r + ng - R) (kRows: s kSR - ng - P) and writes the rows it has exact:
// from its first row in the first strip, to its last in the last one.  The register budget (four
// wavefronts per SIMD, two for a single pass) keeps the compiler from
// computing every row sum of a pass ahead of the radial combinations.
template <class T, int P, int kSR, bool kRows>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P == 1 ? 2 : 4)))
filter_strip_kernel(Grid g, TriT<T> X, CTriT<T> S, int3 half2, int3 parity) {
  constexpr int R = kSR + 2 * P;
  const int lane = (int)threadIdx.x & (kFLanes - 1);
  const int strip = (int)blockIdx.y * 4 + ((int)threadIdx.x >> 6);
  const int nrow = g.n_r + 2 * g.ng;
  if (strip >= filter_strips_r<P, kSR, kRows>(nrow)) return;  // whole wavefront
  int ifirst, rlo, rhi;
  if (kRows) {
    ifirst = strip * kSR - g.ng - P;
    rlo = P;
    rhi = P + kSR;
  } else {
    ifirst = min(strip * kSR - g.ng, g.n_r + g.ng - R);
    rlo = strip == 0 ? 0 : P;
    rhi = ifirst + R >= g.n_r + g.ng ? R : P + kSR;
  }
  const int ld = (int)g.ld, n = g.n_th;
  const int b = (int)blockIdx.x;
  const int Jlo = filter_strip_lo(b, ld);
  const int out_lo = b == 0 ? 0 : Jlo + kFMaxPasses;
  const int out_hi = Jlo + kFLanes >= ld ? ld : Jlo + kFLanes - kFMaxPasses;
  const int J = Jlo + lane, j = J - g.ng;
  const bool col = J < ld, out = col && J >= out_lo && J < out_hi;
  // one component per grid.z (plane pointers selected with scalar code)
  const int c = (int)blockIdx.z;
  const int hs = c == 0 ? half2.x : c == 1 ? half2.y : half2.z;
  T* const x = c == 0 ? X.p[0] : c == 1 ? X.p[1] : X.p[2];
  const T* const sp = c == 0 ? S.p[0] : c == 1 ? S.p[1] : S.p[2];
  FilterAxis ax{};
  const bool axis = filter_strip_axis(b, ld, n, g.ng);  // whole wavefront
  if (axis) {
    ax.hs = hs != 0;
    ax.par = (double)(c == 0 ? parity.x : c == 1 ? parity.y : parity.z);
    ax.lo = j == 0;
    ax.hi = j == n - hs;
    ax.ghost = j < 0 || j > n - hs;
    ax.src = ax.ghost ? lane + axis_mirror(j, n, hs) - j : lane;
  }
  if (axis)
    filter_strip_comp<T, P, kSR, true, kRows>(g, x, sp, J, col, out, ifirst, rlo, rhi, ax);
  else
    filter_strip_comp<T, P, kSR, false, kRows>(g, x, sp, J, col, out, ifirst, rlo, rhi, ax);
}

}  // namespace grpic
