// Device functions shared by the forward flux sweep and its adjoint, so that
// both take the same discrete decisions from the same arithmetic.
#pragma once

#include <math.h>

#include "htr_dev.h"

namespace htr {

// TENO6 cut-off decisions from the four smoothness indicators b_k and the
// global one tau: candidate k is kept when its scale-separated weight
// gamma_k = (1 + tau / (b_k + 1e-40))^6, normalised by the sum over the
// four candidates, reaches C_T.  This is the reference arithmetic (every
// quotient correctly rounded, gamma scaled by the largest r before the
// sixth power); the result is four bits, bit k set when candidate k is kept.
__device__ __forceinline__ unsigned teno6_pattern_exact(double b0, double b1, double b2, double b3, double tau,
                                                        double CT) {
  const double r0 = 1.0 + tau / (b0 + 1e-40), r1 = 1.0 + tau / (b1 + 1e-40);
  const double r2 = 1.0 + tau / (b2 + 1e-40), r3 = 1.0 + tau / (b3 + 1e-40);
  const double irm = 1.0 / fmax(fmax(r0, r1), fmax(r2, r3));
  double g0 = r0 * irm, g1 = r1 * irm, g2 = r2 * irm, g3 = r3 * irm;
  g0 = g0 * g0 * g0; g0 *= g0;
  g1 = g1 * g1 * g1; g1 *= g1;
  g2 = g2 * g2 * g2; g2 *= g2;
  g3 = g3 * g3 * g3; g3 *= g3;
  const double igs = 1.0 / (g0 + g1 + g2 + g3);
  return (g0 * igs >= CT ? 1u : 0u) | (g1 * igs >= CT ? 2u : 0u) | (g2 * igs >= CT ? 4u : 0u) |
         (g3 * igs >= CT ? 8u : 0u);
}

// The same decisions without a correctly rounded quotient.  The test
// gamma_k / sum(gamma) >= C_T is the same as x_k >= C_T sum(x) for x_k =
// (s r_k)^6 with any scale s > 0, here s = 1, so:
//  - the four 1 / (b_k + eps) come from one hardware reciprocal of their
//    product (refined by two Newton steps) and three products each
//    (Montgomery's simultaneous inversion);
//  - each x_k = r_k^6 (r_k >= 1) is then within about 1e-14 (relative) of
//    its exact value, and the reference arithmetic is within about the same
//    distance, so where every x_k lies further than 1e-12 C_T sum(x) from
//    C_T sum(x) both take the same decision.  Otherwise the reference
//    arithmetic decides; so it does for a product of the b_k beyond 1e290,
//    and for an overflow or a non-finite value (the comparison then fails).
// The indicators arrive scaled by 16 (teno6_decide), and so does eps.
__device__ __forceinline__ unsigned teno6_pattern(double b0, double b1, double b2, double b3, double tau,
                                                  double CT) {
  const double D0 = b0 + 16e-40, D1 = b1 + 16e-40, D2 = b2 + 16e-40, D3 = b3 + 16e-40;
  const double P01 = D0 * D1, P23 = D2 * D3, P = P01 * P23;
  double inv = __builtin_amdgcn_rcp(P);
  inv = fma(fma(-P, inv, 1.0), inv, inv);
  inv = fma(fma(-P, inv, 1.0), inv, inv);
  const double i01 = tau * (inv * P23), i23 = tau * (inv * P01);
  double x0 = fma(i01, D1, 1.0), x1 = fma(i01, D0, 1.0);
  double x2 = fma(i23, D3, 1.0), x3 = fma(i23, D2, 1.0);
  x0 = x0 * x0 * x0;
  x1 = x1 * x1 * x1;
  x2 = x2 * x2 * x2;
  x3 = x3 * x3 * x3;
  const double th = CT * fma(x0, x0, fma(x1, x1, fma(x2, x2, x3 * x3)));
  const double y0 = fma(x0, x0, -th), y1 = fma(x1, x1, -th), y2 = fma(x2, x2, -th), y3 = fma(x3, x3, -th);
  const double near = fmin(fmin(fabs(y0), fabs(y1)), fmin(fabs(y2), fabs(y3)));
  if (!(near > 1e-12 * th && P < 1e290))
    return teno6_pattern_exact(0.0625 * b0, 0.0625 * b1, 0.0625 * b2, 0.0625 * b3, 0.0625 * tau, CT);
  // kept: not below the threshold (the sign bits)
  return ((unsigned)~__double2hiint(y0) >> 31) | ((unsigned)~__double2hiint(y1) >> 31) << 1 |
         ((unsigned)~__double2hiint(y2) >> 31) << 2 | ((unsigned)~__double2hiint(y3) >> 31) << 3;
}

// TENO6 cut-off pattern (bit k: candidate k kept) at x_{i+1/2} for one side of
// the Lax-Friedrichs flux splitting, from h[0..5] = 2 f_{i-2..i+3} (the
// splitting's factor 1/2 is folded into the constants).  The smoothness
// indicators and the coefficients of the six-point polynomial are combinations
// of the undivided differences of h (exact rewritings of their sums), 16 times
// their values for f: differences of nearby values are exact, so nearly
// uniform data keep their digits, and with the differences shared the pattern
// takes 55 operations up to tau where the expanded sums take 95.  Cut-offs
// within rounding of CT can fall either way under another arrangement of the
// same sums (as in any arithmetic that isn't the oracle's bit for bit).
__device__ __forceinline__ unsigned teno6_decide(const double h[6], double CT) {
  const double e0 = h[1] - h[0], e1 = h[2] - h[1], e2 = h[3] - h[2], e3 = h[4] - h[3], e4 = h[5] - h[4];
  const double c0 = e1 - e0, c1 = e2 - e1, c2 = e3 - e2, c3 = e4 - e3;
  const double t0 = c1 - c0, t1 = c2 - c1, t2 = c3 - c2;
  const double q0 = t1 - t0, q1 = t2 - t1;
  const double w = q1 - q0;
  const double s = e1 + e2;
  // 16 beta_k: (13/3) (second difference)^2 + (first-order combination)^2
  const double z1 = fma(-2.0, e2, c2), z2 = fma(2.0, e1, c0), z3 = fma(2.0 / 3.0, t2, -z1), s3b = c2 - t2;
  const double b0 = fma((13.0 / 3.0) * c1, c1, s * s);
  const double b1 = fma((13.0 / 3.0) * c2, c2, z1 * z1);
  const double b2 = fma((13.0 / 3.0) * c0, c0, z2 * z2);
  const double b3 = fma((781.0 / 180.0) * t2, t2, fma((13.0 / 3.0) * s3b, s3b, z3 * z3));
  // six-point polynomial (origin at the centre of cell i): 4 a_1, 4 a_2, 12 a_3,
  // 48 a_4 = q0, 240 a_5 = w
  const double v = fma(-0.5, q0, t1);
  const double A1 = fma(259.0 / 2880.0, w, fma(-5.0 / 12.0, v, s));
  const double A2 = fma(-0.125, q0, c1);
  const double A3 = fma(-7.0 / 24.0, w, v);
  double b6 = A1 * fma(1.0 / 480.0, w, fma(1.0 / 6.0, A3, A1));
  b6 = fma(A2, fma(13.0 / 3.0, A2, 0.35 * q0), b6);
  b6 = fma(A3, fma(3129.0 / 720.0, A3, (14127.0 / 40320.0) * w), b6);
  b6 = fma((87617.0 / 20160.0) * q0, q0, b6);
  b6 = fma((252337135.0 / 58060800.0) * w, w, b6);
  const double tau = fabs(fma(-1.0 / 6.0, fma(4.0, b0, b1 + b2), b6));
  return teno6_pattern(b0, b1, b2, b3, tau, CT);
}

// Linear coefficients of the reconstruction that keeps the candidates of a
// cut-off pattern (the normalised weights d_k delta_k / sum d delta with
// d = (9/20, 3/10, 1/20, 1/5)), for f_{i-2..i+3}.
__device__ __forceinline__ void teno6_coeffs_bits(unsigned b, double c[6]) {
  double w0 = (b & 1u) ? 9.0 / 20.0 : 0.0, w1 = (b & 2u) ? 3.0 / 10.0 : 0.0;
  double w2 = (b & 4u) ? 1.0 / 20.0 : 0.0, w3 = (b & 8u) ? 1.0 / 5.0 : 0.0;
  const double iw = 1.0 / (w0 + w1 + w2 + w3);
  w0 *= iw; w1 *= iw; w2 *= iw; w3 *= iw;
  c[0] = w2 * (2.0 / 6.0);
  c[1] = w0 * (-1.0 / 6.0) + w2 * (-7.0 / 6.0);
  c[2] = w0 * (5.0 / 6.0) + w1 * (2.0 / 6.0) + w2 * (11.0 / 6.0) + w3 * (3.0 / 12.0);
  c[3] = w0 * (2.0 / 6.0) + w1 * (5.0 / 6.0) + w3 * (13.0 / 12.0);
  c[4] = w1 * (-1.0 / 6.0) + w3 * (-5.0 / 12.0);
  c[5] = w3 * (1.0 / 12.0);
}

// A block's table of those coefficients for h = 2 f: the reconstruction is
// then six FMAs, whatever the pattern.  Thread t < 16 writes row t; a barrier
// follows before the first use.
__device__ __forceinline__ void teno6_table(unsigned t, double (*tab)[6]) {
  if (t >= 16) return;
  double c[6];
  teno6_coeffs_bits(t, c);
#pragma unroll
  for (int m = 0; m < 6; ++m) tab[t][m] = 0.5 * c[m];
}

// TENO6 reconstruction at x_{i+1/2} of one side of the split with cut-off
// pattern pat, from h = 2 f_{i-2..i+3}.
__device__ __forceinline__ double teno6_value(const double (*tab)[6], unsigned pat, const double h[6]) {
  const double* c = tab[pat];
  return c[0] * h[0] + c[1] * h[1] + c[2] * h[2] + c[3] * h[3] + c[4] * h[4] + c[5] * h[5];
}

// Both sides of the split: the TENO6 face flux.
__device__ __forceinline__ double teno6_face(const double (*tab)[6], const double hp[6], const double hm[6],
                                             double CT) {
  return teno6_value(tab, teno6_decide(hp, CT), hp) + teno6_value(tab, teno6_decide(hm, CT), hm);
}

// Third-order WENO-Z reconstruction at x_{i+1/2} (Don & Borges) from f_{i-1},
// f_i, f_{i+1} = f[1..3] of the six-point face stencil: candidates on
// {i-1, i} and {i, i+1} with optimal weights 1/3 and 2/3, smoothness the
// squared first differences, global indicator |beta_0 - beta_1|.
__device__ __forceinline__ double weno3z(const double f[6]) {
  const double q0 = (-f[1] + 3.0 * f[2]) / 2.0;
  const double q1 = (f[2] + f[3]) / 2.0;
  const double b0 = (f[2] - f[1]) * (f[2] - f[1]);
  const double b1 = (f[3] - f[2]) * (f[3] - f[2]);
  const double tau = fabs(b0 - b1);
  const double a0 = (1.0 / 3.0) * (1.0 + tau / (b0 + 1e-40));
  const double a1 = (2.0 / 3.0) * (1.0 + tau / (b1 + 1e-40));
  return (a0 * q0 + a1 * q1) / (a0 + a1);
}

// WENO3-Z of one side of the split from h = 2 f (the stencil values halved
// first, as the scheme takes them).
__device__ __forceinline__ double weno3z_h(const double h[6]) {
  double f[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) f[m] = 0.5 * h[m];
  return weno3z(f);
}

// Node convective flux of variable v along d (u_d normal velocity, p pressure).
template <int NS>
__device__ __forceinline__ double node_flux(int v, int d, double U, double ud, double p) {
  if (v == NS + 3) return (U + p) * ud;
  if (v == NS + d) return U * ud + p;
  return U * ud;
}

__device__ __forceinline__ double hRTi(const MechTables* __restrict__ M, int s, double T, double iT) {
  const double* a = M->hc[s];
  return a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4]))) + a[5] * iT;
}

}  // namespace htr
