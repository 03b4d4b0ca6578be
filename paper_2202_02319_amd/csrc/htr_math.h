// Device arithmetic shared by the per-cell kernel and its adjoint: short
// exponentials and reciprocals, and the tabulated collision integral.
#pragma once

#include <math.h>

#include "htr_dev.h"

namespace htr {

// exp(x) for |x| up to 1e6 (2^n saturates to 0 or infinity): x = n ln 2 + r, |r| <= ln 2 / 2, and
// exp(r) = 1 + r + r^2 q(r), q the degree-9 interpolant of (exp(r) - 1 - r) / r^2
// at Chebyshev nodes (remainder 2e-17).  18 vector instructions; the general
// library function spends about ten more on the ends of the range.
__device__ __forceinline__ double exp_in(double x) {
  const double n = rint(x * 1.4426950408889634074);
  double r = fma(n, -0.69314718055994530942, x);
  r = fma(n, -2.3190468138462995584e-17, r);
  double q = 2.510038549551032e-08;
  q = fma(q, r, 2.7620088445409746e-07);
  q = fma(q, r, 2.7557268459997064e-06);
  q = fma(q, r, 2.4801521295954376e-05);
  q = fma(q, r, 0.00019841269863053618);
  q = fma(q, r, 0.0013888888917213717);
  q = fma(q, r, 0.008333333333330062);
  q = fma(q, r, 0.04166666666662413);
  q = fma(q, r, 0.16666666666666669);
  q = fma(q, r, 0.5000000000000001);
  return __builtin_ldexp(1.0 + fma(r * r, q, r), (int)n);
}

// The same for any x (0 and infinity at the ends, infinity for NaN: a rate
// constant's two sides then give NaN).
__device__ __forceinline__ double exp_sat(double x) { return exp_in(fmax(fmin(x, 1e4), -1e4)); }

// 1/x and 1/sqrt(x) of normal positive x: the hardware estimate and two
// Newton steps (the last residual is formed with one rounding, so the result
// is within an ulp).
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-(x * y), y, 1.0), y);
  return fma(0.5 * y, fma(-(x * y), y, 1.0), y);
}

// Stages a table (om11 or its derivative) in LDS; a barrier follows.
__device__ __forceinline__ void stage_om(double* to, const double (*from)[OMDEG + 1], int rows) {
  const double2* f = reinterpret_cast<const double2*>(from);
  double2* t = reinterpret_cast<double2*>(to);
  for (int k = threadIdx.x; k < rows * (OMDEG + 1) / 2; k += blockDim.x) t[k] = f[k];
}

// The species pairs i < j.
template <int NS>
struct Pairs {
  static constexpr int N = NS * (NS - 1) / 2;
  int i[N + 1] = {}, j[N + 1] = {};
  constexpr Pairs() {
    int p = 0;
    for (int a = 0; a < NS; ++a)
      for (int b = a + 1; b < NS; ++b, ++p) {
        i[p] = a;
        j[p] = b;
      }
  }
};
constexpr int OMPF = 3;
// Neufeld-Janzen-Aziz collision integral Omega11(T*): from the staged table
// (row = the top bits of T*, a polynomial in T* - the interval's centre), or
// the fit itself, pw = T*^(-0.1561) its power (a product of a factor per cell and
// one per pair).  The table's eight coefficients are four 16-byte LDS reads and
// seven FMAs where the fit takes three exponentials.
template <bool TAB>
__device__ __forceinline__ double omega11(const double* __restrict__ s_om, int row0, int rows, double Ts, double pw) {
  if constexpr (TAB) {
    const int hi = __double2hiint(Ts);
    const unsigned row = min((unsigned)((hi >> 15) - row0), (unsigned)(rows - 1));
    const double t = Ts - __hiloint2double((hi & (int)0xffff8000) | 0x4000, 0);
    const double* c = s_om + row * (OMDEG + 1);
    double v = c[OMDEG];
#pragma unroll
    for (int k = OMDEG - 1; k >= 0; --k) v = fma(v, t, c[k]);
    return v;
  } else {
    return 1.06036 * pw + 0.19300 * exp(-0.47635 * Ts) + 1.03587 * exp(-1.52996 * Ts) + 1.76474 * exp(-3.89411 * Ts);
  }
}

}  // namespace htr
