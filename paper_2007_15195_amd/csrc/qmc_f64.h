// FP64 QMC kernels: steps a4-a5 of a Vecchia term (Section 2.2, eq. (6)) in
// double precision, for FP64 evaluations and for the terms an FP32 evaluation
// hands over. Per chain (variables 0..k, the term's own component last):
//     e_0 = Phi(b_0 / L_00)                   (constant, from term_setup)
//     y_{a-1} = Phi^{-1}(w_{a-1} e_{a-1})      a = 1..k
//     t_a = b'_a - sum_{c<a} L'_ac y_c,   e_a = Phi(t_a)
//     den = prod_{a<s} e_a (1 for s = 0),   num = prod_{a<=k} e_a
// with s = k for a plain term and the term's split for a joint block term
// (Section 3.2). One wave runs one work item, points across its 64 lanes.
//
// K is the most steps a kernel runs, a template parameter, so that the chain is
// unrolled and y[] stays in registers; a term with k < K leaves the chain after
// step k (a scalar compare per step).
//
// What bounds it: the FP64 vector unit (one wave instruction per CU-clock), so
// the step is written for few instructions. The normal CDF and quantile are
// nearest-node Taylor polynomials from tables in LDS (device_nodes_f64.h),
// loaded once per workgroup: 2 x 12 CU-clocks of LDS gathers run beside about
// 75 of arithmetic. The fitted ratios (out of line) take over only where a lane
// leaves the tables' ranges (q < 2^-15 or t < -8.5; about 1% of wave-steps at
// thresholds near the 0.9 quantile). The term's rows come through scalar loads
// as scalar operands, which cost an FP64 FMA nothing, while LDS broadcasts took
// 2.4 clocks of the LDS pipe per coefficient and 8-49 KB per wave.
// Measured against one-wave workgroups with the fitted ratios, rows in LDS and,
// above 31 steps, y in LDS: 2,500 terms, k = 10, 10^4 x 10 points 17.3 -> 5.4 ms
// (4.6e11 steps/s, 86 CU-clocks a wave-step); 900 terms, k = 50, 3607 x 10 points
// 76.9 -> 8.5 ms; 10,000 FP32 terms with k = 30 of which many run again in FP64
// 25.3 -> 16.6 ms.
// A workgroup holds W waves with their own items, and two workgroups fit a
// compute unit's LDS (64 KB of tables each); W is 8, 6 or 4, the most waves
// (4, 3 or 2 per SIMD) whose registers hold 2K doubles without spilling.
#pragma once
#include <utility>

#include "vecchia_internal.h"

#include "device_math_f64.h"
#include "device_nodes_f64.h"
#include "lattice.h"
#include "qmc_items.h"

namespace vecchia {
namespace {

// Constant address space: uniform reads become scalar loads.
using ScalarRows = const __attribute__((address_space(4))) double*;
using ScalarGen = const __attribute__((address_space(4))) uint64_t*;

// The fitted functions, out of line: the rare lanes outside the tables.
__device__ __noinline__ double ncdf64(double t) { return phi64(t); }
__device__ __noinline__ double ncdfinv64(double u) { return ninv64(u); }

// Waves per workgroup: two workgroups per compute unit.
constexpr int f64_waves(int K) { return K <= 32 ? 8 : K <= 52 ? 6 : 4; }
// Chains up to this many steps advance U_j in registers (one add per step);
// longer ones form p Z_j + S_j from shifts staged in LDS, which frees 2K registers.
constexpr int kF64AdvanceK = 12;

__device__ __forceinline__ void load_nodes(double* nodes) {
  const double2* src = reinterpret_cast<const double2*>(kNormNodeTable);
  double2* dst = reinterpret_cast<double2*>(nodes);
  for (int e = threadIdx.x; e < kNormNodes; e += blockDim.x) dst[e] = src[e];
  __syncthreads();
}

// State of one lane's chain over the unrolled steps.
template <int K>
struct Chain64 {
  double y[K];
  double e, prod, head;
  uint64_t dead;   // lanes whose chain reached a factor 0 (or NaN)
};

// Step A and, through the recursion, the steps after it up to min(k, K).
template <int A, int K>
__device__ __forceinline__ void steps_f64(Chain64<K>& s, uint64_t* U, const uint64_t* sh, ScalarGen Z, ScalarRows rows,
                                          const double* nodes, int k, int sp, uint32_t pt) {
  if (A > k) return;
  if (A == sp) {
    __asm__ volatile("");   // a scalar branch, not a select in every step
    s.head = s.prod;
  }
  uint64_t Ua;
  if constexpr (K <= kF64AdvanceK) {
    Ua = U[A - 1];
    U[A - 1] += Z[A - 1] << 6;
  } else {
    Ua = (uint64_t)pt * Z[A - 1] + sh[A - 1];
  }
  const double w = lattice_coord_f64(Ua);
  // y = Phi^{-1}(u) from q = min(u, 1 - u) (1 - u is exact for u >= 1/2)
  double u, uc, side;
  {
    // the product rounds before 1 - u, as the quantile's argument is u itself
#pragma clang fp contract(off)
    u = w * s.e;
    uc = 1.0 - u;
    side = u - 0.5;
  }
  const double q = fmin(u, uc);
  double ya = __builtin_copysign(ninv_nodes(nodes, q), side);
  if (__builtin_expect(any_lane(!(q >= kNinvNodeMin)), 0)) {
    if (!(q >= kNinvNodeMin)) ya = s.e > 0.0 ? ncdfinv64(fmax(u, 2.2250738585072014e-308)) : 0.0;
    s.dead = __builtin_amdgcn_ballot_w64(!(s.e > 0.0));
  }
  s.y[A - 1] = ya;
  const ScalarRows row = rows + A * (A + 1) / 2;
  double t = row[A];
#pragma unroll
  for (int c = 0; c < A; ++c) t -= row[c] * s.y[c];
  double e = phi_nodes(nodes, fmax(fmin(t, kPhiNodeMax), -kPhiNodeMax));
  if (__builtin_expect((__builtin_amdgcn_ballot_w64(!(t >= -kPhiNodeMax)) | s.dead) != 0, 0)) {
    if (!(t >= -kPhiNodeMax)) e = ncdf64(t);
    if ((s.dead >> (threadIdx.x & 63)) & 1) e = 0.0;
  }
  s.e = e;
  {
    // no contraction: num takes the rounded products that den takes
#pragma clang fp contract(off)
    s.prod = s.prod * e;
  }
  if constexpr (A < K) steps_f64<A + 1, K>(s, U, sh, Z, rows, nodes, k, sp, pt);
}

// One item by the calling wave. rows: the term's FP64 rows (row a at a (a + 1) / 2);
// sh: K shifts of the wave (K > kF64AdvanceK).
template <int K>
__device__ __forceinline__ void item_f64(const Item& it, const Aux64* __restrict__ aux64, const uint64_t* __restrict__ Zg,
                                         double* __restrict__ sums, const double* __restrict__ rows_g,
                                         const double* nodes, uint64_t* sh) {
  const InstDesc& I = *it.I;
  const int lane = threadIdx.x & 63;
  int k = it.K;
  int sp = I.split ? uniform(I.split[it.i]) : k;
  const double e0 = aux64[it.t].e0;
  const int p_begin = 1 + it.c * I.chunk_points;
  const int p_last = min(I.n_points, p_begin + I.chunk_points - 1);
  uintptr_t Z_u = (uintptr_t)Zg;
  constexpr bool kAdvance = K <= kF64AdvanceK;
  uint64_t U[kAdvance ? K : 1];
  if constexpr (kAdvance) {
    const ScalarGen Z = (ScalarGen)Z_u;
#pragma unroll
    for (int j = 0; j < K; ++j)
      U[j] = (uint64_t)(p_begin + lane) * Z[j] + lattice_shift(I.seed, it.i, it.sr, j, it.second);
  } else {
    for (int j = lane; j < k; j += 64) sh[j] = lattice_shift(I.seed, it.i, it.sr, j, it.second);
    __builtin_amdgcn_wave_barrier();   // the wave's own slice: written and read in program order
  }
  double acc_num = 0.0, acc_den = 0.0;
  uintptr_t rows_u = (uintptr_t)rows_g;
  for (int p0 = p_begin; p0 <= p_last; p0 += 64) {
    // opaque per iteration: rows and generators are loaded where a step uses
    // them instead of all being held (and spilled) across the point loop
    // (k and sp likewise: compared in place, not held as 2K lane masks)
    __asm__ volatile("" : "+s"(rows_u), "+s"(Z_u), "+s"(k), "+s"(sp)::"memory");
    Chain64<K> s;
    s.e = e0;
    s.prod = e0;
    s.head = 1.0;
    s.dead = 0;
    steps_f64<1, K>(s, U, sh, (ScalarGen)Z_u, (ScalarRows)rows_u, nodes, k, sp, (uint32_t)(p0 + lane));
    if (p0 + lane <= p_last) {
#pragma clang fp contract(off)
      acc_den += s.head;
      acc_num += s.prod;
    }
  }
  acc_num = wave_sum(acc_num);
  acc_den = wave_sum(acc_den);
  if (lane == 0) {
    double* o = item_out(I, it, sums);
    o[0] = acc_num;
    o[1] = acc_den;
    o[2] = -1.0;
  }
}

// The workgroup in slot g of the grid (xcd_slot) takes the W items_per_wave consecutive items from
// g W items_per_wave on, its waves one after another.
template <int K>
__global__ __launch_bounds__(64 * f64_waves(K)) __attribute__((amdgpu_waves_per_eu(f64_waves(K) / 2))) void qmc_f64(
    const InstDesc* __restrict__ insts, const RangeDesc* __restrict__ ranges, int n_ranges,
    const Aux64* __restrict__ aux64, const uint64_t* __restrict__ Zg, double* __restrict__ sums, int64_t item_base,
    int64_t item_end, int items_per_wave, int even) {
  constexpr int W = f64_waves(K);
  __shared__ __align__(16) double nodes[2 * kNormNodes];
  __shared__ uint64_t sh[K > kF64AdvanceK ? W * K : 1];
  load_nodes(nodes);
  const int wv = uniform(threadIdx.x >> 6);
  int64_t g = item_base + (int64_t)xcd_slot(blockIdx.x, gridDim.x, even != 0) * (int64_t)(W * items_per_wave) + wv;
  for (int j = 0; j < items_per_wave && g < item_end; ++j, g += W) {
    const Item it = decode_item(insts, ranges, n_ranges, g);
    item_f64<K>(it, aux64, Zg, sums, reinterpret_cast<const double*>(it.I->prep) + it.i * it.I->prep_stride, nodes,
                sh + (K > kF64AdvanceK ? wv * K : 0));
  }
}

__device__ __forceinline__ int find_inst_q(const int64_t* __restrict__ bases, int n, int64_t t) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (bases[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Handed-over terms of FP32 instances, from both lists: each wave takes the next
// (list entry, item) pair from the work counter ctr[1] until the counts x ipt_max
// pairs are used up; pairs past a term's own item count are skipped. Every wave leaves
// once the counter passes the end, so the grid always drains. K covers every
// term of the batch's FP32 instances.
template <int K>
__global__ __launch_bounds__(64 * f64_waves(K)) __attribute__((amdgpu_waves_per_eu(f64_waves(K) / 2))) void qmc_promoted(
    const InstDesc* __restrict__ insts, int n_inst, const int64_t* __restrict__ term_bases,
    const Aux64* __restrict__ aux64, const uint64_t* __restrict__ Zg, double* __restrict__ sums,
    const int32_t* __restrict__ list, int64_t* __restrict__ ctr, int64_t cap, int ipt_max) {
  constexpr int W = f64_waves(K);
  __shared__ __align__(16) double nodes[2 * kNormNodes];
  __shared__ uint64_t sh[K > kF64AdvanceK ? W * K : 1];
  const int64_t first = min(ctr[0], cap);
  const int64_t total = (first + min(ctr[2], cap)) * (int64_t)ipt_max;
  if ((int64_t)blockIdx.x * W >= total) return;   // fewer pairs than waves: no tables, no work counter
  load_nodes(nodes);
  const int lane = threadIdx.x & 63, wv = uniform(threadIdx.x >> 6);
  for (;;) {
    // The taker's predicate is opaque and behind a convergent barrier: on the
    // plain lane == 0, which also guards the item's store at the end of the
    // loop, the optimizer threads the two branches together, so that the other
    // lanes loop apart from lane 0, read their own got = 0 and never leave.
    int taker = lane;
    __asm__ volatile("" : "+v"(taker));
    __builtin_amdgcn_wave_barrier();
    unsigned long long got = 0;
    if (taker == 0) got = atomicAdd(reinterpret_cast<unsigned long long*>(&ctr[1]), 1ULL);
    __builtin_amdgcn_wave_barrier();
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)got);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(got >> 32));
    const int64_t v = (int64_t)(((uint64_t)hi << 32) | lo);
    if (v >= total) break;
    const int64_t e = v / ipt_max;
    const int j = (int)(v - e * ipt_max);
    const int64_t t = uniform(list[e < first ? e : cap + (e - first)]);
    const int ii = uniform(find_inst_q(term_bases, n_inst, t));
    const InstDesc& I = insts[ii];
    const int ns = uniform(I.n_shifts), nc = uniform(I.n_chunks);
    if (j >= uniform(I.passes) * ns * nc) continue;
    Item it;
    it.I = &I;
    it.i = t - term_bases[ii];
    it.t = t;
    it.r = j / nc;
    it.c = j - it.r * nc;
    it.second = it.r >= ns;
    it.sr = it.second ? it.r - ns : it.r;
    it.K = uniform(I.sovk[it.i]);
    item_f64<K>(it, aux64, Zg, sums, prep_f64(I, it.i), nodes, sh + (K > kF64AdvanceK ? wv * K : 0));
  }
}

template <int K>
hipError_t launch_f64_k(const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                        const Aux64* aux64, const uint64_t* Z, double* sums, hipStream_t s) {
  constexpr int W = f64_waves(K);
  // items per wave: enough to repay a workgroup's table load (about 2 us) while
  // every compute unit still gets four rounds of workgroups
  const int64_t most = K < 64 ? 64 / K : 1;
  int64_t per = (span.end - span.begin) / ((int64_t)W * 2048);
  per = per < 1 ? 1 : per > most ? most : per;
  const int64_t block_items = W * per;
  const int64_t max_blocks = kMaxLaunchThreads / (64 * W);
  for (int64_t b = span.begin; b < span.end; b += max_blocks * block_items) {
    const int64_t left = (span.end - b + block_items - 1) / block_items;
    const unsigned n = (unsigned)(left < max_blocks ? left : max_blocks);
    hipLaunchKernelGGL(qmc_f64<K>, dim3(n), dim3(64 * W), 0, s, insts, ranges, n_ranges, aux64, Z, sums, b, span.end,
                       (int)per, (int)span.even);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int K>
hipError_t launch_promoted_k(const InstDesc* insts, int n_inst, const int64_t* term_bases, const Aux64* aux64,
                             const uint64_t* Z, double* sums, const int32_t* list, int64_t* ctr, int64_t cap,
                             int ipt_max, hipStream_t s) {
  constexpr int W = f64_waves(K);
  const int64_t blocks = (cap * (int64_t)ipt_max + W - 1) / W;
  const unsigned grid = (unsigned)(blocks < 512 ? blocks : 512);   // two workgroups per compute unit
  hipLaunchKernelGGL(qmc_promoted<K>, dim3(grid), dim3(64 * W), 0, s, insts, n_inst, term_bases, aux64, Z, sums, list,
                     ctr, cap, ipt_max);
  return hipGetLastError();
}

// The launch of the kernel for kc steps, among the sizes SizeOf(0), SizeOf(1), ...
template <int (*SizeOf)(int), int... Is>
hipError_t run_f64(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                   const Aux64* aux64, const uint64_t* Z, double* sums, hipStream_t s, std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == SizeOf(Is) ? (e = launch_f64_k<SizeOf(Is)>(insts, ranges, n_ranges, span, aux64, Z, sums, s), 0) : 0), ...);
  return e;
}

template <int (*SizeOf)(int), int... Is>
hipError_t run_promoted(int kc, const InstDesc* insts, int n_inst, const int64_t* term_bases, const Aux64* aux64,
                        const uint64_t* Z, double* sums, const int32_t* list, int64_t* ctr, int64_t cap, int ipt_max,
                        hipStream_t s, std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == SizeOf(Is)
        ? (e = launch_promoted_k<SizeOf(Is)>(insts, n_inst, term_bases, aux64, Z, sums, list, ctr, cap, ipt_max, s), 0)
        : 0),
   ...);
  return e;
}

}  // namespace
}  // namespace vecchia
