// Small device-side helpers shared by the rate kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace eph {

template <class T>
struct V2;
template <>
struct V2<double> {
  using t = double2;
};
template <>
struct V2<float> {
  using t = float2;
};

template <class T>
__device__ __forceinline__ typename V2<T>::t mk(T x, T y) {
  typename V2<T>::t r;
  r.x = x;
  r.y = y;
  return r;
}

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

// (a mod N) for |a| < 2^31, result in [0, N)
__device__ __forceinline__ int imod(int a, int N) {
  int r = a % N;
  return r < 0 ? r + N : r;
}

// exp(x) for x <= 0 by Cody and Waite's reduction x = n ln 2 + r (ln 2 as a
// 32-bit head and a tail) and the Taylor series of e^r to r^13 (|r| <= 0.347:
// remainder below 5e-18), scaled by 2^n.  No special values to tell apart, so
// 19 instructions.
__host__ __device__ __forceinline__ double exp_neg(double x) {
  x = fmax(x, -800.0);
  const double n = rint(x * 1.4426950408889634074);
  double r = fma(n, -6.93147180369123816490e-01, x);  // head of ln 2, then its tail
  r = fma(n, -1.90821492927058770002e-10, r);
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, (int)n);
}

// (r, i) += a * b with four fused multiply-adds
template <class T>
__device__ __forceinline__ void cmac(T &r, T &i, T ar, T ai, T br, T bi) {
  r = fma(ar, br, r);
  r = fma(-ai, bi, r);
  i = fma(ar, bi, i);
  i = fma(ai, br, i);
}
// (r, i) += conj(a) * b
template <class T>
__device__ __forceinline__ void cmac_conj(T &r, T &i, T ar, T ai, T br, T bi) {
  r = fma(ar, br, r);
  r = fma(ai, bi, r);
  i = fma(ar, bi, i);
  i = fma(-ai, br, i);
}

}  // namespace eph
