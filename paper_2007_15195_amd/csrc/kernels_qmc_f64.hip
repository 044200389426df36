// FP64 QMC kernels for chains of up to 32 steps (qmc_f64.h).
#include "qmc_f64.h"

namespace vecchia {
namespace {

// Kernel sizes: 2, 4, ..., 32; a chain of k steps runs in the next size up.
constexpr int size_of(int i) { return 2 * i + 2; }

}  // namespace

hipError_t launch_qmc_f64_short(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                                const Aux64* aux64, const uint64_t* Z, double* sums, hipStream_t s) {
  return run_f64<size_of>(kc, insts, ranges, n_ranges, span, aux64, Z, sums, s, std::make_integer_sequence<int, 16>{});
}

hipError_t launch_qmc_promoted_short(int kc, const InstDesc* insts, int n_inst, const int64_t* term_bases,
                                     const Aux64* aux64, const uint64_t* Z, double* sums, const int32_t* list,
                                     int64_t* ctr, int64_t cap, int ipt_max, hipStream_t s) {
  return run_promoted<size_of>(kc, insts, n_inst, term_bases, aux64, Z, sums, list, ctr, cap, ipt_max, s,
                               std::make_integer_sequence<int, 16>{});
}

}  // namespace vecchia
