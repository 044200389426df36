// FP32 QMC kernels for joint block terms (qmc_f32.h).
#include "qmc_f32.h"

namespace vecchia {
namespace {

// Kernel sizes: 4, 8, ..., 60, 63; a chain of k steps runs in the next size up.
constexpr int size_of(int i) { return f32_block_kernel_size(4 * i + 1); }

}  // namespace

hipError_t launch_qmc_f32_block(int kc, const InstDesc* insts, const RangeDesc* ranges, int n_ranges, ItemSpan span,
                                const Aux32* aux32, const uint64_t* Z, double* sums, hipStream_t s) {
  return run_f32<size_of, true>(kc, insts, ranges, n_ranges, span, aux32, Z, sums, s,
                                std::make_integer_sequence<int, 16>{});
}

}  // namespace vecchia
