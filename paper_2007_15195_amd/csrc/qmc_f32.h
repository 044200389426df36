// FP32 QMC kernels: steps a4-a5 of a Vecchia term (Section 2.2, eq. (6); Genz's
// separation of variables with a randomized lattice rule) in single precision.
// Per chain (variables 0..k, the term's own component last):
//     e_0 = Phi(b'_0)                         (constant, from term_setup)
//     y_{a-1} = Phi^{-1}(w_{a-1} e_{a-1})      a = 1..k
//     t_a = b'_a - sum_{c<a} L'_ac y_c,   e_a = Phi(t_a)
//     den = prod_{a<k} e_a,    num = den * e_k
// (the constant e_0 cancels from the ratio and is left out of these products).
// Joint block terms (Section 3.2; the BLOCK variants) keep every factor in the
// product instead and take the denominator at the term's split s:
//     den = prod_{a<s} e_a (1 for s = 0),   num = prod_{a<=k} e_a,
// with 1 - prod_{a>=s} e_a carried as its own recurrence for the log1p form.
// The wave writes {sum num, sum den, sum den*(1-e_k)} of its chunk, summed over
// lanes by a fixed butterfly, so an item's result does not depend on where or
// with what else it runs.
//
// What bounds it: the vector unit, and there the instruction kinds. Measured in
// CU-clocks per wave instruction on gfx950: an FP32 FMA, add or multiply and a
// two-operand integer operation take 0.55-0.6 from vector registers or with a
// literal, 1.08 with a scalar register; compares, selects, conversions, min and
// three-operand integer operations 1.0; exp, log, rcp and sqrt 2.0. An LDS
// broadcast of 16 bytes takes 4.3 clocks of the LDS pipe, a 16-byte gather from
// the quantile's cells 12, both beside the vector unit. So a step
//  * takes the quantile from a table in LDS, one quadratic per 1/32 octave of
//    q (2.9 clocks; log, sqrt, a ratio and its reciprocal took 16);
//  * takes Phi(-|t|) as 2^p(|v|), a polynomial with literal coefficients (7.3;
//    the ratio, its reciprocal and an exponential took 11 to 14);
//  * forms u = w e and 1 - u as em - wc em and m + wc em (wc = 1 - w), two FMAs
//    whose smaller result is the quantile's argument;
//  * has one rare-case test: a quantile argument below 2^-15, which every
//    factor below 2^-15 implies in the next step. Such lanes take the
//    previous factor and the quantile again in the accurate split form below.
// Measured over whole launches (8192 x 8 points, thresholds at 1.28), CU-clocks a
// step now and with one-wave workgroups, fitted ratios and rows in LDS:
// k = 10: 27.0 (38.8); k = 20: 31.8 (43.1); k = 31: 39.8 (56.7); k = 63: 57.7 (147).
//
// Rare lanes (cold32, cold32_first; 0.7% of wave-steps with thresholds near the
// 0.9 quantile, 3% to 15% with rough thresholds on a smooth field, counted by the
// 72 vector instructions that such a step adds): factors are
// e = em * 2^en, with en = 0 except for a rare lane's lower-tail factors, which
// keep 2^floor(-v^2) in en so that em stays in [R, 2R). The product of the factors is
// qm * 2^qe (qe an integer): a common factor is at least 2^-15, so qm is
// renormalised every fourth step where it fell below 2^-50, and around every
// rare step; it never leaves the normal range. The last factor of a chain, whose
// complement the log1p form needs to full relative accuracy, always takes the
// ratio of phi_f32.
//
// K is the most steps a kernel runs, a template parameter, so that the chain is
// unrolled and y[] stays in registers; a term with k < K leaves the chain after
// step k (a scalar compare per step). The term's scaled rows come through scalar
// loads as scalar operands: 1.05 clocks a coefficient, where LDS broadcasts took
// 0.6 on the vector unit and 1.2 on the LDS pipe beside the table's gathers, 2.1
// measured. (Two points per lane, sharing LDS row reads, take the coefficients'
// cost down to 0.6 and the whole step not at all: 27.8 clocks against 27.0.) A
// workgroup is four waves with their own items around one table (8 KB), eight
// workgroups to a compute unit.
#pragma once
#include <utility>

#include "vecchia_internal.h"

#include "device_math_f32.h"
#include "lattice.h"
#include "normal_tables_f32.h"
#include "qmc_items.h"

namespace vecchia {
namespace {

constexpr int kF32Waves = 4;
constexpr float kDeepV = 7.74596669f;      // sqrt(60)
constexpr float kQuantMin = 0x1p-15f;      // the table's range: q in [2^-15, 1/2]
constexpr int kQuantSlots = 512;           // any exponent and mantissa address one of these
// Chains up to this many steps advance U_j in registers (one add per step);
// longer ones form p Z_j + S_j from shifts staged in LDS, which frees 2K registers.
constexpr int kF32AdvanceK = 24;
// Waves per SIMD to fit: the most whose registers hold the chain.
constexpr int f32_min_waves(int K) { return K <= 12 ? 8 : K <= 18 ? 6 : K <= 24 ? 5 : K <= 32 ? 6 : K <= 48 ? 5 : 4; }

using ScalarGen32 = const __attribute__((address_space(4))) uint64_t*;
using ScalarRows32 = const __attribute__((address_space(4))) float*;

// p * a + literal, the coefficient in the instruction. No operand may come straight from exp, log, rcp or sqrt: the wait state that
// gfx950 wants behind those is not inserted before inline assembly.
#define VECCHIA_FMAAK(p, a, k)                                                                                      \
  __asm__("v_fmaak_f32 %0, %1, %2, %3" : "=v"(p) : "v"(p), "v"(a), "i"(__builtin_bit_cast(uint32_t, (float)(k))))

// Phi(-|v| / kappa) for |v| <= 3.41 (Phi >= 2^-15), with a relative error below
// 0.9e-6 for |v| < 0.5, rising to 1.8e-6 at 3.4 (the fit's 0.8e-6 and the rounding
// of an exponent near -15), 5.6e-7 in the mean square; beyond it falls to 0 with an
// absolute error below 5e-11. (The (3,4) ratio before: 1.4e-6 and 6.7e-7. A
// polynomial of degree 10 has 1.3e-6 and 2.0e-7 for two more instructions a step;
// one of degree 9 rises beyond the range; other weights at degree 8 take the 1.8e-6
// down to 1.4e-6 and the error for |v| < 1, where most factors lie, up by a third.)
__device__ __forceinline__ float tail_f32(float v) {
  const float a = fabsf(v);
  float p = kTailPoly[8];
  VECCHIA_FMAAK(p, a, kTailPoly[7]);
  VECCHIA_FMAAK(p, a, kTailPoly[6]);
  VECCHIA_FMAAK(p, a, kTailPoly[5]);
  VECCHIA_FMAAK(p, a, kTailPoly[4]);
  VECCHIA_FMAAK(p, a, kTailPoly[3]);
  VECCHIA_FMAAK(p, a, kTailPoly[2]);
  VECCHIA_FMAAK(p, a, kTailPoly[1]);
  VECCHIA_FMAAK(p, a, kTailPoly[0]);
  return fast_exp2(p);
}

// R = erfcx(|t| / sqrt 2) / 2, t = v / kappa, with f = -v^2. |v| enters capped at
// 2^24: beyond, where a nearly singular block scales a limit by up to 1e8, the
// denominator's a^5 would overflow and its reciprocal make R zero and the next
// quantile NaN. The exponent f, which stops at -2^20, decides the value there.
__device__ __forceinline__ float ratio_f32(float v, float* f) {
  const float a = fminf(fabsf(v), 0x1p24f);
  *f = -(v * v);
  float p = kRP[4], q = kRQ[5];
  VECCHIA_FMAAK(p, a, kRP[3]);
  VECCHIA_FMAAK(p, a, kRP[2]);
  VECCHIA_FMAAK(p, a, kRP[1]);
  VECCHIA_FMAAK(p, a, kRP[0]);
  VECCHIA_FMAAK(q, a, kRQ[4]);
  VECCHIA_FMAAK(q, a, kRQ[3]);
  VECCHIA_FMAAK(q, a, kRQ[2]);
  VECCHIA_FMAAK(q, a, kRQ[1]);
  VECCHIA_FMAAK(q, a, kRQ[0]);
  return p * fast_rcp(q);
}
// Phi(t) from v = kappa t, as e = em (exact unless em is split further by the
// caller) with the smaller tail m = Phi(-|t|) = 2^f R, f = -v^2.
struct PhiParts {
  float em;   // Phi(t)
  float m;    // Phi(-|t|)
  float f;    // -v^2
  float R;    // erfcx(|t| / sqrt 2) / 2
  bool neg;   // t <= 0
};
__device__ __forceinline__ PhiParts phi_f32(float v) {
  PhiParts o;
  o.R = ratio_f32(v, &o.f);
  o.m = fast_exp2(o.f) * o.R;
  o.neg = v <= 0.0f;
  o.em = o.neg ? o.m : 1.0f - o.m;
  return o;
}

// The cells to LDS, by a workgroup of kThreads.
template <int kThreads>
__device__ __forceinline__ void load_cells(float4* cells) {
  for (int e = threadIdx.x; e < kQuantSlots; e += kThreads)
    cells[e] = reinterpret_cast<const float4*>(kQuantTable)[e < kQuantCells ? e : kQuantCells - 1];
  __syncthreads();
}

// -Phi^{-1}(q) from the cells, absolute error below 4e-7; any q outside their range
// addresses some slot.
__device__ __forceinline__ float quant_f32(const float4* cells, float q) {
  const uint32_t off = (__builtin_bit_cast(uint32_t, q) >> 14) & 0x1ff0u;
  const float4 c = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(cells) + off);
  const float d = q - c.w;
  return fmaf(fmaf(c.z, d, c.y), d, c.x);
}

struct Cold32 {
  float em, en, y;   // the previous factor em * 2^en and -Phi^{-1}(w em 2^en)
};

// A rare lane's step: the previous factor from its v, and the quantile of w times
// it. A lower-tail factor keeps 2^floor(-v^2) in en (bounded, so that the sum of
// exponents cannot overflow). Out of line: inlined it is 3% faster where a fifth
// of the wave-steps are rare and k = 20, and 2.5% slower at k = 50.
__device__ __noinline__ Cold32 cold32(float v, float awc) {
  float f, R = ratio_f32(v, &f);
  f = f < -1048576.0f ? -1048576.0f : f;   // a NaN stays
  const float fl = floorf(f);
  const float mm = fast_exp2(f - fl) * R;
  const bool neg = v <= 0.0f;
  const float m = ldexpf(mm, (int)fl);
  Cold32 o;
  o.em = neg ? mm : 1.0f - m;
  o.en = neg ? fl : 0.0f;
  const float um = fmaf(-awc, o.em, o.em);
  const bool lower = neg || um <= 0.5f;
  const float z = ninv_tail_from_log2_split(fast_log2(lower ? um : fmaf(awc, o.em, m)) + o.en);
  o.y = lower ? z : -z;
  return o;
}

// The same for the first step, whose factor is term_setup's e_0 = em 2^en.
__device__ __noinline__ float cold32_first(float em, float en, float ec, bool neg, float awc) {
  const float um = fmaf(-awc, em, em);
  const bool lower = neg || um <= 0.5f;
  const float z = ninv_tail_from_log2_split(fast_log2(lower ? um : fmaf(awc, em, ec)) + en);
  return lower ? z : -z;
}

template <int K>
struct Chain32 {
  float y[K];      // -y (the recursion then adds, in the short FMA encoding)
  float em, m;     // the latest factor and 1 - it (or Phi(-|t|))
  float v;         // its argument, kappa t
  float qm;        // product of factors, qm 2^qe
  int qe;
  float dm;        // BLOCK: prod_{a<s} e_a = dm 2^de
  int de;
  float cc;        // BLOCK: 1 - prod_{s<=a} e_a so far
};

// Step A and, through the recursion, the steps after it; returns with v_k.
template <int A, int K, bool BLOCK>
__device__ __forceinline__ void steps_f32(Chain32<K>& s, uint64_t* U, const uint64_t* sh, ScalarGen32 Z, ScalarRows32 rows,
                                          const float4* cells, float c24, const Aux32& ax, bool split0, int k, int sp,
                                          uint32_t pt) {
  uint32_t hi;
  if constexpr (K <= kF32AdvanceK) {
    hi = (uint32_t)(U[A - 1] >> 32);
    U[A - 1] += Z[A - 1] << 6;
  } else {
    hi = (uint32_t)(((uint64_t)pt * Z[A - 1] + sh[A - 1]) >> 32);
  }
  const float wc = lattice_complement_f32(hi, c24);    // 1 - w
  const float um = fmaf(-wc, s.em, s.em);              // u = w e
  const float qt = fminf(um, fmaf(wc, s.em, s.m));     // min(u, 1 - u)
  float y = __builtin_copysignf(quant_f32(cells, qt), 0.5f - um);
  bool rare = !(qt >= kQuantMin);
  if (A == 1) rare = rare || split0;
  if (__builtin_expect(any_lane(rare), 0)) {
    if constexpr (A == 1) {
      if (rare) y = cold32_first(ax.em0, ax.en0, ax.ec0, ax.neg0 != 0.0f, wc);
    } else {
      s.qe += __builtin_amdgcn_frexp_expf(s.qm);
      s.qm = __builtin_amdgcn_frexp_mantf(s.qm);
      if (rare) {
        const Cold32 c = cold32(s.v, wc);
        s.em = c.em;
        s.qe += (int)c.en;
        y = c.y;
      }
    }
  }
  s.y[A - 1] = y;
  if constexpr (A >= 2) {
    s.qm *= s.em;
    if constexpr (A % 4 == 0) {
      if (__builtin_expect(any_lane(s.qm < 0x1p-50f), 0)) {
        s.qe += __builtin_amdgcn_frexp_expf(s.qm);
        s.qm = __builtin_amdgcn_frexp_mantf(s.qm);
      }
    }
  }
  if (BLOCK && A == sp) {
    __asm__ volatile("");   // a scalar branch, not selects in every step
    s.dm = s.qm;
    s.de = s.qe;
  }
  constexpr int ro = A * (A + 1) / 2;
  float v = rows[ro + A];
#pragma unroll
  for (int c = 0; c < A; ++c) v = fmaf(rows[ro + c], s.y[c], v);
  s.v = v;
  if constexpr (A < K) {
    if (A == k) return;
    if (BLOCK && A >= sp) {
      // a factor of the numerator's tail: its complement to full relative accuracy
      const PhiParts ph = phi_f32(v);
      s.em = ph.em;
      s.m = ph.m;
      s.cc = fmaf(ph.neg ? 1.0f - ph.em : ph.m, 1.0f - s.cc, s.cc);
    } else {
      s.m = tail_f32(v);
      s.em = v <= 0.0f ? s.m : 1.0f - s.m;
    }
    steps_f32<A + 1, K, BLOCK>(s, U, sh, Z, rows, cells, c24, ax, split0, k, sp, pt);
  }
}

template <int K, bool BLOCK>
__device__ __forceinline__ void item_f32(const Item& it, const Aux32* __restrict__ aux32, const uint64_t* __restrict__ Zg,
                                         double* __restrict__ sums, uint64_t* sh, const float4* cells) {
  const InstDesc& I = *it.I;
  if (uniform(I.promote[it.t]) != 0) return;   // this term runs in FP64 (qmc_promoted)
  const int lane = threadIdx.x & 63;
  int k = it.K;
  int sp = BLOCK ? uniform(I.split[it.i]) : k;   // denominator: the first sp factors
  const float* __restrict__ prep = reinterpret_cast<const float*>(I.prep) + it.i * I.prep_stride;
  const Aux32 ax = aux32[it.t];
  const bool split0 = uniform(ax.en0 != 0.0f) != 0;
  const int p_begin = 1 + it.c * I.chunk_points;
  const int p_last = min(I.n_points, p_begin + I.chunk_points - 1);
  uintptr_t Z_u = (uintptr_t)Zg;
  constexpr bool kAdvance = K <= kF32AdvanceK;
  uint64_t U[kAdvance ? K : 1];
  if constexpr (kAdvance) {
    // the lane's chain starts at point p_begin + lane and strides 64: U_j += 64 Z_j
    const ScalarGen32 Z = (ScalarGen32)Z_u;
#pragma unroll
    for (int j = 0; j < K; ++j)
      U[j] = (uint64_t)(p_begin + lane) * Z[j] + lattice_shift(I.seed, it.i, it.sr, j, it.second);
  } else {
    for (int j = lane; j < k; j += 64) sh[j] = lattice_shift(I.seed, it.i, it.sr, j, it.second);
  }
  uintptr_t rows_u = (uintptr_t)prep;
  __builtin_amdgcn_wave_barrier();          // the wave's own LDS slice: program order suffices
  float c24 = 0x1p-24f;
  __asm__ volatile("" : "+v"(c24));
  double acc_num = 0.0, acc_den = 0.0, acc_cnum = 0.0;
  for (int p0 = p_begin; p0 <= p_last; p0 += 64) {
    // opaque per iteration: the rows and generators come through scalar loads
    // where a step uses them instead of being held across the loop, and k and sp
    // are compared in place
    __asm__ volatile("" : "+s"(Z_u), "+s"(rows_u), "+s"(k), "+s"(sp)::"memory");
    Chain32<K> s;
    s.em = ax.em0;
    s.m = ax.ec0;
    s.qm = 1.0f;
    s.qe = 0;
    s.dm = 1.0f;
    s.de = 0;
    s.cc = 0.0f;
    if (BLOCK) {
      // every factor is in the products, e_0 included
      s.qe = (int)ax.en0 + __builtin_amdgcn_frexp_expf(ax.em0);
      s.qm = __builtin_amdgcn_frexp_mantf(ax.em0);
      if (sp == 0) s.cc = ax.ec0;
    }
    steps_f32<1, K, BLOCK>(s, U, sh, (ScalarGen32)Z_u, (ScalarRows32)rows_u, cells, c24, ax, split0, k, sp, (uint32_t)(p0 + lane));
    // the last factor, to full accuracy; its exponent and the product's are 0
    // but for rare lanes
    const PhiParts ph = phi_f32(s.v);
    double em = (double)ph.em, ec = (double)(ph.neg ? 1.0f - ph.em : ph.m);
    double den = (double)(BLOCK ? s.dm : s.qm), num = (double)s.qm;
    const uint64_t odd = __builtin_amdgcn_ballot_w64(s.v < -kDeepV) | __builtin_amdgcn_ballot_w64((s.qe | s.de) != 0);
    if (__builtin_expect(odd != 0, 0)) {
      if (s.v < -kDeepV) {
        const float f = fmaxf(ph.f, -1048576.0f), fl = floorf(f);
        em = ldexp((double)(fast_exp2(f - fl) * ph.R), (int)fl);
        ec = 1.0 - em;
      }
      den = ldexp(den, BLOCK ? s.de : s.qe);
      num = ldexp(num, s.qe);
    }
    if (p0 + 63 > p_last && p0 + lane > p_last) den = num = 0.0;   // past the chunk's last point
    acc_den += den;
    if (BLOCK) {
      ec = (double)fmaf((float)ec, 1.0f - s.cc, s.cc);
      acc_num = fma(num, em, acc_num);
    } else {
      acc_num = fma(den, em, acc_num);
    }
    acc_cnum = fma(den, ec, acc_cnum);
  }
  acc_num = wave_sum(acc_num);
  acc_den = wave_sum(acc_den);
  acc_cnum = wave_sum(acc_cnum);
  if (lane == 0) {
    double* o = item_out(I, it, sums);
    o[0] = acc_num;
    o[1] = acc_den;
    o[2] = acc_cnum;
  }
}

// The workgroup in slot g of the grid (xcd_slot) takes the 4 items_per_wave consecutive items from
// 4 items_per_wave g on, its waves one after another.
template <int K, bool BLOCK>
__global__ __launch_bounds__(64 * kF32Waves) __attribute__((amdgpu_waves_per_eu(f32_min_waves(K)))) void qmc_f32(
    const InstDesc* __restrict__ insts, const RangeDesc* __restrict__ ranges, int n_ranges,
    const Aux32* __restrict__ aux32, const uint64_t* __restrict__ Zg, double* __restrict__ sums, int64_t item_base,
    int64_t item_end, int items_per_wave, int even) {
  __shared__ float4 cells[kQuantSlots];
  __shared__ uint64_t sh[kF32Waves][K > kF32AdvanceK ? K : 1];
  load_cells<64 * kF32Waves>(cells);
  const int wv = uniform(threadIdx.x >> 6);
  int64_t g = item_base + (int64_t)xcd_slot(blockIdx.x, gridDim.x, even != 0) * (int64_t)(kF32Waves * items_per_wave) + wv;
  for (int j = 0; j < items_per_wave && g < item_end; ++j, g += kF32Waves) {
    const Item it = decode_item(insts, ranges, n_ranges, g);
    item_f32<K, BLOCK>(it, aux32, Zg, sums, sh[wv], cells);
  }
}

template <int K, bool BLOCK>
hipError_t launch_f32_k(const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                        const Aux32* aux32, const uint64_t* Z, double* sums, hipStream_t s) {
  // items per wave: up to 4 repay a workgroup's table load (8 KB, about 1 us)
  // while every compute unit still gets four rounds of workgroups
  int64_t per = (span.end - span.begin) / ((int64_t)kF32Waves * 8192);
  per = per < 1 ? 1 : per > 4 ? 4 : per;
  const int64_t block_items = kF32Waves * per;
  constexpr int64_t kMaxBlocks = kMaxLaunchThreads / (64 * kF32Waves);
  for (int64_t b = span.begin; b < span.end; b += kMaxBlocks * block_items) {
    const int64_t left = (span.end - b + block_items - 1) / block_items;
    const unsigned n = (unsigned)(left < kMaxBlocks ? left : kMaxBlocks);
    hipLaunchKernelGGL((qmc_f32<K, BLOCK>), dim3(n), dim3(64 * kF32Waves), 0, s, insts, ranges, n_ranges, aux32, Z, sums,
                       b, span.end, (int)per, (int)span.even);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The launch of the kernel for kc steps, among the sizes SizeOf(0), SizeOf(1), ...
template <int (*SizeOf)(int), bool BLOCK, int... Is>
hipError_t run_f32(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                   const Aux32* aux32, const uint64_t* Z, double* sums, hipStream_t s, std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == SizeOf(Is) ? (e = launch_f32_k<SizeOf(Is), BLOCK>(insts, ranges, n_ranges, span, aux32, Z, sums, s), 0) : 0), ...);
  return e;
}

}  // namespace
}  // namespace vecchia
