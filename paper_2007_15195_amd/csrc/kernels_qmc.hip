// QMC launches: steps a4-a5 of every Vecchia term (Section 2.2, eq. (6); Genz's
// separation of variables with a randomized lattice rule).
//
// Work item = (term, pass, shift, chunk): one wave evaluates one chunk of the N
// lattice points of one random shift of one term, points across the 64 lanes. A
// launch runs the smallest kernel built for its longest chains: qmc_f32.h (FP32 evaluations) and
// qmc_f64.h (FP64 evaluations, and the terms an FP32 evaluation hands over).
#include "vecchia_internal.h"

namespace vecchia {

hipError_t launch_qmc(int K, int precision, bool block, const InstDesc* d_insts, const RangeDesc* d_ranges,
                      int n_ranges, ItemSpan span, const Aux64* aux64, const Aux32* aux32,
                      const uint64_t* d_Z, double* sums, hipStream_t s) {
  if (span.end <= span.begin) return hipSuccess;
  if (K < 1 || K > kMaxM || span.begin < 0 || span.end > 0x7fffffffLL) return hipErrorInvalidValue;
  const int kc = qmc_kernel_size(K);
  if (precision == VECCHIA_FP64)
    return kc <= kQmcShortK ? launch_qmc_f64_short(kc, d_insts, d_ranges, n_ranges, span, aux64, d_Z, sums, s)
                            : launch_qmc_f64_long(kc, d_insts, d_ranges, n_ranges, span, aux64, d_Z, sums, s);
  if (block)
    return launch_qmc_f32_block(f32_block_kernel_size(K), d_insts, d_ranges, n_ranges, span, aux32, d_Z, sums, s);
  return kc <= kQmcShortK ? launch_qmc_f32_short(kc, d_insts, d_ranges, n_ranges, span, aux32, d_Z, sums, s)
                          : launch_qmc_f32_long(kc, d_insts, d_ranges, n_ranges, span, aux32, d_Z, sums, s);
}

hipError_t launch_qmc_promoted(int K, const InstDesc* d_insts, int n_inst, const int64_t* d_term_bases,
                               const Aux64* aux64, const uint64_t* d_Z, double* sums, const int32_t* list,
                               int64_t* ctr, int64_t cap, int ipt_max, hipStream_t s) {
  if (cap <= 0 || ipt_max <= 0 || K <= 0) return hipSuccess;
  if (K > kMaxM) return hipErrorInvalidValue;
  const int kc = qmc_kernel_size(K);
  return kc <= kQmcShortK
             ? launch_qmc_promoted_short(kc, d_insts, n_inst, d_term_bases, aux64, d_Z, sums, list, ctr, cap, ipt_max, s)
             : launch_qmc_promoted_long(kc, d_insts, n_inst, d_term_bases, aux64, d_Z, sums, list, ctr, cap, ipt_max, s);
}

}  // namespace vecchia
