// FP64 QMC kernels for chains of 33 to 63 steps (qmc_f64.h).
#include <utility>

#include "qmc_f64.h"

namespace vecchia {
namespace {

constexpr int f64_long_kc(int i) { return i < 15 ? 34 + 2 * i : kMaxM; }

// Kernel sizes kc = 34, 36, ..., 62, 63: a chain of k steps runs in the next size up.
template <int... Is>
hipError_t run_f64(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                   const Aux64* aux64, const uint64_t* Z, double* sums, hipStream_t s,
                   std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == f64_long_kc(Is) ? (e = launch_f64_k<f64_long_kc(Is)>(insts, ranges, n_ranges, span, aux64, Z, sums, s), 0) : 0), ...);
  return e;
}

template <int... Is>
hipError_t run_promoted(int kc, const InstDesc* insts, int n_inst, const int64_t* term_bases, const Aux64* aux64,
                        const uint64_t* Z, double* sums, const int32_t* list, int64_t* ctr, int64_t cap, int ipt_max,
                        hipStream_t s, std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == f64_long_kc(Is) ? (e = launch_promoted_k<f64_long_kc(Is)>(insts, n_inst, term_bases, aux64, Z, sums, list, ctr, cap, ipt_max, s), 0) : 0),
   ...);
  return e;
}

}  // namespace

hipError_t launch_qmc_f64_long(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                          const Aux64* aux64, const uint64_t* Z, double* sums, hipStream_t s) {
  return run_f64(kc, insts, ranges, n_ranges, span, aux64, Z, sums, s, std::make_integer_sequence<int, 16>{});
}

hipError_t launch_qmc_promoted_long(int kc, const InstDesc* insts, int n_inst, const int64_t* term_bases,
                               const Aux64* aux64, const uint64_t* Z, double* sums, const int32_t* list,
                               int64_t* ctr, int64_t cap, int ipt_max, hipStream_t s) {
  return run_promoted(kc, insts, n_inst, term_bases, aux64, Z, sums, list, ctr, cap, ipt_max, s,
                      std::make_integer_sequence<int, 16>{});
}

}  // namespace vecchia
