// FP64 normal CDF and quantile of the QMC loops from node tables held in LDS
// (normal_tables.h): the nearest node's value and a Taylor polynomial about it.
// Every derivative is a polynomial in the node, so a node is two doubles, one
// 16-byte LDS read per evaluation.
//
// Quantile, q in [2^-15, 1/2]: with q_i the midpoint of q's cell (128 cells per
// octave), z_i = -Phi^{-1}(q_i) and x = (q_i - q) / phi(z_i),
//     z = z_i + x + z x^2/2 + (2 z^2 + 1) x^3/6 + (6 z^3 + 7 z) x^4/24
//         + (24 z^4 + 46 z^2 + 7) x^5/120 + (120 z^5 + 326 z^3 + 127 z) x^6/720   (z = z_i on the right),
// the inverse function's series (dz/dx = phi(z_i) / phi(z)). |x| <= 2^-8 / z, so the first term
// left out is below 2^-58 z.
// CDF, |t| <= 8.5: with a_i the nearest multiple of 1/128 and d = t - a_i,
//     Phi(t) = Phi(a_i) + phi(a_i) d [1 + sum_{k=1..6} (-1)^k He_k(a_i) d^k / (k + 1)!],
// He_k the Hermite polynomials (by their recurrence, which needs few constants). The first term left out is below 2^-54 Phi(t).
// Both are within 2.1e-16 relative of 40-digit values over their ranges (the
// quantile at q -> 1/2, where z -> 0, within 2^-60 absolute), against 5.5e-16
// and 7.6e-16 of the fitted ratios of device_math_f64.h, which remain the
// functions outside these ranges.
//
// About 20 FP64 instructions each and no branch inside, where the ratios take
// 150 (quantile: a division, a logarithm, a square root and two of its three
// pieces in nearly every wave) and 66 (CDF).
#pragma once

#include <cstdint>
#include <cstring>

#include "normal_tables.h"

namespace vecchia {

constexpr double kNinvNodeMin = 0x1p-15;   // quantile nodes: q in [2^-15, 1/2]
constexpr double kPhiNodeMax = 8.5;        // CDF nodes: |t| <= 8.5 (1 beyond it above)

__host__ __device__ __forceinline__ uint64_t bits_of(double x) {
  uint64_t b;
  __builtin_memcpy(&b, &x, 8);
  return b;
}
__host__ __device__ __forceinline__ double of_bits(uint64_t b) {
  double x;
  __builtin_memcpy(&x, &b, 8);
  return x;
}

// z = -Phi^{-1}(q), q in [2^-15, 1/2]; any other q reads some node below
// byte 32768 of the table and returns garbage.
__host__ __device__ __forceinline__ double ninv_nodes(const double* nodes, double q) {
  const uint32_t hi = (uint32_t)(bits_of(q) >> 32);
  // exponent's low 4 bits and 7 mantissa bits: 2^-15 is entry 0
  const double* nd = reinterpret_cast<const double*>(reinterpret_cast<const char*>(nodes) + ((hi >> 9) & 0x7ff0u));
  const double z = nd[0], r = nd[1];
  const double qi = of_bits((uint64_t)((hi & 0xffffe000u) | 0x1000u) << 32);
  const double x = (qi - q) * r;
  // z2 and a2 below enter with a source modifier: without one the compiler
  // takes the two-operand FMA and copies each constant into a vector register
  const double z2 = __builtin_fabs(z * z);
  const double c3 = __builtin_fma(__builtin_fabs(z2), 1.0 / 3.0, 1.0 / 6.0);
  const double c4 = z * __builtin_fma(__builtin_fabs(z2), 0.25, 7.0 / 24.0);
  const double c5 = __builtin_fma(__builtin_fabs(z2), __builtin_fma(__builtin_fabs(z2), 0.2, 46.0 / 120.0), 7.0 / 120.0);
  const double c6 = z * __builtin_fma(__builtin_fabs(z2), __builtin_fma(__builtin_fabs(z2), 1.0 / 6.0, 326.0 / 720.0),
                                      127.0 / 720.0);
  double p = __builtin_fma(x, c6, c5);
  p = __builtin_fma(x, p, c4);
  p = __builtin_fma(x, p, c3);
  p = __builtin_fma(x, p, 0.5 * z);
  p = __builtin_fma(x, p, 1.0);
  return __builtin_fma(x, p, z);
}

// Phi(t), |t| <= 8.5 (the caller clamps).
__host__ __device__ __forceinline__ double phi_nodes(const double* nodes, double t) {
  constexpr double kRound = 0x1.8p45;   // t + kRound rounds t to a multiple of 2^-7, held in the low bits
  const double s = t + kRound;
  const double a = s - kRound;
  const int i = (int)(uint32_t)bits_of(s);
  const double* nd = nodes + 2 * kNinvNodes + 2 * (i + kPhiMid);
  const double P = nd[0], f = nd[1];
  const double d = t - a;
  // g_k = (-d)^k He_k(a): g_{k+1} = -(a d) g_k - k d^2 g_{k-1}
  const double u = a * d, v = d * d;
  const double g2 = __builtin_fma(u, u, -v);
  const double g3 = -u * __builtin_fma(-2.0, v, g2);
  const double g4 = __builtin_fma(-u, g3, -__builtin_fma(2.0, v, v) * g2);
  const double g5 = __builtin_fma(-u, g4, -4.0 * v * g3);
  const double g6 = __builtin_fma(-u, g5, -__builtin_fma(4.0, v, v) * g4);
  double p = __builtin_fma(u, -0.5, 1.0);
  p = __builtin_fma(g2, 1.0 / 6.0, p);
  p = __builtin_fma(g3, 1.0 / 24.0, p);
  p = __builtin_fma(g4, 1.0 / 120.0, p);
  p = __builtin_fma(g5, 1.0 / 720.0, p);
  p = __builtin_fma(g6, 1.0 / 5040.0, p);
  return __builtin_fma(f * d, p, P);
}

}  // namespace vecchia
