// tangent.hpp -- FP64 value with N directional derivatives (forward-mode
// tangents), for the position derivatives of the metric in the adjoint.  The
// templated metric code of geometry.hpp runs on it unchanged.
#pragma once

#include "geometry.hpp"

namespace grpic {

template <int N>
struct Tan {
  double v;
  double d[N];
  Tan() = default;
  __host__ __device__ Tan(double x) : v(x) {  // a constant: zero tangents
#pragma unroll
    for (int k = 0; k < N; ++k) d[k] = 0.0;
  }
};
template <int N>
struct ScalarOf<Tan<N>> {
  using type = double;
};

template <int N>
__device__ inline Tan<N> operator+(const Tan<N>& a, const Tan<N>& b) {
  Tan<N> r;
  r.v = a.v + b.v;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = a.d[k] + b.d[k];
  return r;
}
template <int N>
__device__ inline Tan<N> operator-(const Tan<N>& a, const Tan<N>& b) {
  Tan<N> r;
  r.v = a.v - b.v;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = a.d[k] - b.d[k];
  return r;
}
template <int N>
__device__ inline Tan<N> operator-(const Tan<N>& a) {
  Tan<N> r;
  r.v = -a.v;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = -a.d[k];
  return r;
}
template <int N>
__device__ inline Tan<N> operator*(const Tan<N>& a, const Tan<N>& b) {
  Tan<N> r;
  r.v = a.v * b.v;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = a.d[k] * b.v + a.v * b.d[k];
  return r;
}
// with a constant: no operations on its zero tangents
template <int N>
__device__ inline Tan<N> operator*(double a, const Tan<N>& b) {
  Tan<N> r;
  r.v = a * b.v;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = a * b.d[k];
  return r;
}
template <int N>
__device__ inline Tan<N> operator*(const Tan<N>& a, double b) {
  return b * a;
}
template <int N>
__device__ inline Tan<N> operator+(const Tan<N>& a, double b) {
  Tan<N> r = a;
  r.v = a.v + b;
  return r;
}
template <int N>
__device__ inline Tan<N> operator+(double a, const Tan<N>& b) {
  return b + a;
}
template <int N>
__device__ inline Tan<N> operator-(const Tan<N>& a, double b) {
  Tan<N> r = a;
  r.v = a.v - b;
  return r;
}
template <int N>
__device__ inline Tan<N> operator-(double a, const Tan<N>& b) {
  Tan<N> r = -b;
  r.v = a - b.v;
  return r;
}
// x -> f(x) with f' = df at the value
template <int N>
__device__ inline Tan<N> chain(const Tan<N>& a, double f, double df) {
  Tan<N> r;
  r.v = f;
#pragma unroll
  for (int k = 0; k < N; ++k) r.d[k] = df * a.d[k];
  return r;
}
template <int N>
__device__ inline Tan<N> rcp(const Tan<N>& a) {
  const double y = rcp(a.v);
  return chain(a, y, -y * y);
}
template <int N>
__device__ inline Tan<N> rsqrt(const Tan<N>& a) {
  const double y = rsqrt(a.v);
  return chain(a, y, -0.5 * y * (y * y));
}

}  // namespace grpic
