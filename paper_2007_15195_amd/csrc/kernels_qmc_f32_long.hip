// FP32 QMC kernels for plain chains of 33 to 63 steps (qmc_f32.h).
#include "qmc_f32.h"

namespace vecchia {
namespace {

// Kernel sizes: 34, 36, ..., 62, 63; a chain of k steps runs in the next size up.
constexpr int size_of(int i) { return i < 15 ? 34 + 2 * i : kMaxM; }

}  // namespace

hipError_t launch_qmc_f32_long(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                                const Aux32* aux32, const uint64_t* Z, double* sums, hipStream_t s) {
  return run_f32<size_of, false>(kc, insts, ranges, n_ranges, span, aux32, Z, sums, s,
                                std::make_integer_sequence<int, 16>{});
}

}  // namespace vecchia
