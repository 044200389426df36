// Work items of the QMC kernels: (term, pass, shift, chunk), one wave each.
#pragma once
#include "vecchia_internal.h"
#include "xcd_map.h"

namespace vecchia {

__device__ __forceinline__ int find_range(const RangeDesc* __restrict__ r, int n, int64_t g) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (r[mid].item_begin <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// true when the predicate holds on some active lane (the ballot's mask is a
// scalar, so the result is wave-uniform)
__device__ __forceinline__ bool any_lane(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

struct Item {
  const InstDesc* I;
  int64_t i;      // plan index of the term
  int64_t t;      // global term index
  int r;          // pass * n_shifts + shift: the item's slot among the term's shifts
  int sr;         // shift
  bool second;    // pass 1: the term's second lattice (independent-points estimator)
  int c;          // chunk
  int K;
};

__device__ __forceinline__ Item decode_item(const InstDesc* __restrict__ insts,
                                            const RangeDesc* __restrict__ ranges, int n_ranges,
                                            int64_t g) {
  const int ri = uniform(find_range(ranges, n_ranges, g));
  const RangeDesc& R = ranges[ri];
  const int local = uniform((int)(g - R.item_begin));      // < 2^31 per range
  const int ipt = R.items_per_term;
  const int term_off = uniform(local / ipt);
  const int rem = local - term_off * ipt;
  Item it;
  it.I = insts + R.inst;
  it.i = R.term_begin + term_off;
  it.r = uniform(rem / R.n_chunks);
  it.c = uniform(rem - it.r * R.n_chunks);
  const int ns = uniform(it.I->n_shifts);
  it.second = it.r >= ns;
  it.sr = it.second ? it.r - ns : it.r;
  it.K = uniform(R.K);
  it.t = it.I->term_base + it.i;
  return it;
}

__device__ __forceinline__ double* item_out(const InstDesc& I, const Item& it, double* sums) {
  return sums + 3 * (I.sums_base + (it.i * I.passes * I.n_shifts + it.r) * (int64_t)I.n_chunks + it.c);
}

}  // namespace vecchia
