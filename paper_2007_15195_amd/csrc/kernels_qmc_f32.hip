// FP32 QMC kernels for plain chains of up to 32 steps (qmc_f32.h).
#include <utility>

#include "qmc_f32.h"

namespace vecchia {
namespace {

// Kernel sizes: 2, 4, ..., 32; a chain of k steps runs in the next size up.
constexpr int size_of(int i) { return 2 * i + 2; }

template <int... Is>
hipError_t run(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span, const Aux32* aux32,
               const uint64_t* Z, double* sums, hipStream_t s, std::integer_sequence<int, Is...>) {
  hipError_t e = hipErrorInvalidValue;
  ((kc == size_of(Is)
        ? (e = launch_f32_k<size_of(Is), false>(insts, ranges, n_ranges, span, aux32, Z, sums, s), 0)
        : 0),
   ...);
  return e;
}

}  // namespace

hipError_t launch_qmc_f32_short(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                          const Aux32* aux32, const uint64_t* Z, double* sums, hipStream_t s) {
  return run(kc, insts, ranges, n_ranges, span, aux32, Z, sums, s, std::make_integer_sequence<int, 16>{});
}

}  // namespace vecchia
