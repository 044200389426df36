// Test hooks: the device's own normal CDF / quantile pieces and lattice points,
// evaluated elementwise on caller data, so that tests can pin them directly
// against library routines and the exact integer lattice definition. Nothing
// here is on the evaluation path.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device_math_f64.h"
#include "device_nodes_f64.h"
#include "lattice.h"
#include "qmc_f32.h"
#include "runtime.h"
#include "vecchia.h"

namespace vecchia {
namespace {

constexpr int kProbeThreads = 256;

// what (see vecchia_probe_math): out has 3 doubles per input
__global__ __launch_bounds__(kProbeThreads) void probe_math(int what, int64_t n, const double* __restrict__ in,
                                                            double* __restrict__ out) {
  __shared__ float4 cells[kQuantSlots];
  load_cells<kProbeThreads>(cells);
  const int64_t i = (int64_t)blockIdx.x * kProbeThreads + threadIdx.x;
  if (i >= n) return;
  const double x = in[i];
  const float v = (float)(x * kPhiScale);   // the FP32 loop's argument kappa t at t = x
  double o0 = 0.0, o1 = 0.0, o2 = 0.0;
  if (what == VECCHIA_PROBE_PHI_F32) {
    // the smaller tail as a chain's last factor has it, and as the rare path splits it
    o0 = phi_f32(v).m;
    const Cold32 c = cold32(-fabsf(v), 0.5f);
    o1 = c.em;
    o2 = c.en;
  } else if (what == VECCHIA_PROBE_TAIL_F32) {
    o0 = tail_f32(v);
  } else if (what == VECCHIA_PROBE_RARE_F32) {
    const Cold32 c = cold32(v, 0.5f);
    o0 = c.y;
    o1 = c.em;
    o2 = c.en;
  } else if (what == VECCHIA_PROBE_NINV_F32) {
    // from its cell, below the cells from log2 q
    const float q = (float)x;
    o0 = q >= kQuantMin ? quant_f32(cells, q) : ninv_tail_from_log2_split(fast_log2(q));
    o1 = q;
  } else if (what == VECCHIA_PROBE_NINV_LOG2_F32) {
    o0 = ninv_tail_from_log2_split((float)x);
  } else if (what == VECCHIA_PROBE_PHI_F64) {
    // as the FP64 loop: the node table, the fitted ratio below it
    o0 = x >= -kPhiNodeMax ? phi_nodes(kNormNodeTable, fmin(x, kPhiNodeMax)) : phi64(x);
  } else {
    // (the loop's value at exactly 1/2 is 1.2e-18, the fitted ratio's is 0)
    const double q = fmin(x, 1.0 - x);
    o0 = q >= kNinvNodeMin && q < 0.5 ? copysign(ninv_nodes(kNormNodeTable, q), x - 0.5) : ninv64(x);
  }
  out[3 * i] = o0;
  out[3 * i + 1] = o1;
  out[3 * i + 2] = o2;
}

__global__ __launch_bounds__(kProbeThreads) void probe_lattice(const uint64_t* __restrict__ Z, uint64_t seed,
                                                               int64_t term, int r, int dim, int second, int64_t n,
                                                               double* __restrict__ w64, float* __restrict__ w32) {
  const int64_t i = (int64_t)blockIdx.x * kProbeThreads + threadIdx.x;
  if (i >= n) return;
  const uint64_t U = (uint64_t)(i + 1) * Z[dim] + lattice_shift(seed, term, r, dim, second != 0);
  if (w64) w64[i] = lattice_coord_f64(U);
  if (w32) w32[i] = 1.0f - lattice_complement_f32((uint32_t)(U >> 32), 0x1p-24f);
}

}  // namespace
}  // namespace vecchia

extern "C" {

vecchia_status vecchia_probe_math(int32_t what, int64_t n, const double* in_dev, double* out_dev,
                                  void* hip_stream) {
  using namespace vecchia;
  if (what < VECCHIA_PROBE_PHI_F32 || what > VECCHIA_PROBE_RARE_F32)
    return set_error(VECCHIA_E_INVALID, "unknown probe");
  if (n < 0 || n > (1LL << 30)) return set_error(VECCHIA_E_INVALID, "n must be in 0..2^30");
  if (n == 0) return VECCHIA_OK;
  if (!in_dev || !out_dev) return set_error(VECCHIA_E_INVALID, "null pointer");
  const unsigned blocks = (unsigned)((n + kProbeThreads - 1) / kProbeThreads);
  hipLaunchKernelGGL(probe_math, dim3(blocks), dim3(kProbeThreads), 0, static_cast<hipStream_t>(hip_stream), what,
                     n, in_dev, out_dev);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "probe launch");
  return VECCHIA_OK;
}

vecchia_status vecchia_probe_lattice(uint64_t seed, int64_t term, int32_t shift, int32_t dim, int32_t second,
                                     int64_t n, double* w64_dev, float* w32_dev, void* hip_stream) {
  using namespace vecchia;
  if (term < 0 || term >= (1LL << 31) || shift < 0 || shift >= VECCHIA_MAX_SHIFTS || dim < 0 || dim >= kMaxM ||
      (second != 0 && second != 1))
    return set_error(VECCHIA_E_INVALID, "term, shift, dim or second out of range");
  if (n < 0 || n > (1LL << 30)) return set_error(VECCHIA_E_INVALID, "n must be in 0..2^30");
  if (n == 0) return VECCHIA_OK;
  if (!w64_dev && !w32_dev) return set_error(VECCHIA_E_INVALID, "no output");
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_error(e, "device query");
  const uint64_t* Z = device_lattice_table(dev, &e);
  if (!Z) return hip_error(e, "lattice table");
  const unsigned blocks = (unsigned)((n + kProbeThreads - 1) / kProbeThreads);
  hipLaunchKernelGGL(probe_lattice, dim3(blocks), dim3(kProbeThreads), 0, static_cast<hipStream_t>(hip_stream), Z,
                     seed, term, shift, dim, second, n, w64_dev, w32_dev);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "probe launch");
  return VECCHIA_OK;
}

}  // extern "C"
