// Randomized Richtmyer lattice points (device side).
//
// Generator z_j = frac(sqrt(p_j)), p_j the j-th prime, held as the 64-bit
// fixed-point integer Z_j (computed on the host by an exact integer square
// root and passed to the kernels). Shift S = SplitMix64 output number
// n = (term << 21) | (shift << 5) | dim (dim < 32) of the stream seeded with
// the call's seed (Steele, Lea & Flood 2014). Point p: U = p Z_j + S mod 2^64; baker
// transform W = |2U - 2^64| (2^64 saturates); the coordinate is the midpoint
// of W's cell on the 2^-52 grid (FP64) or, from U's upper half, on the 2^-23
// grid (FP32).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace vecchia {

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t n) {
  uint64_t z = seed + (n + 1) * 0x9E3779B97F4A7C15ULL;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Dimensions 32..62 (terms of more than 32 variables) take the key
// 2^62 + (term << 22) + (shift << 6) + dim, a range the first form never reaches.
// A term's second lattice (the denominators of the independent-points
// estimator) adds 2^61 to the key: no first-lattice key has that bit set.
__device__ __forceinline__ uint64_t lattice_shift(uint64_t seed, int64_t term, int r, int dim, bool second) {
  const uint64_t salt = second ? (1ULL << 61) : 0ULL;
  if (dim < 32) return splitmix64(seed, salt | ((uint64_t)term << 21) | ((uint64_t)r << 5) | (uint64_t)dim);
  return splitmix64(seed, salt | (1ULL << 62) | ((uint64_t)term << 22) | ((uint64_t)r << 6) | (uint64_t)dim);
}

// FP64 coordinate (2 floor(W / 2^12) + 1) 2^-53, W = |2U - 2^64| (2^64 saturates).
// With V = U for U >= 2^63 and V = U - 1 below (so that U = 0 joins the upper
// half, where it saturates) and f = floor((V mod 2^63) / 2^11) 2^-52, placed in
// the mantissa of 1 + f, the coordinate is t = f + 2^-53 in the upper half and
// 1 - t in the lower; every operation is exact.
__device__ __forceinline__ double lattice_coord_f64(uint64_t U) {
  const int32_t lower = (int32_t)~(uint32_t)(U >> 32) >> 31;   // -1 for U < 2^63, else 0
  const uint64_t V = U + (uint64_t)(int64_t)lower;
  const uint32_t vh = (uint32_t)(V >> 32);
  const uint32_t mh = ((vh >> 11) & 0xfffffu) | 0x3ff00000u;
  const uint32_t ml = __builtin_amdgcn_alignbit(vh, (uint32_t)V, 11);
  const double t = __longlong_as_double((long long)(((uint64_t)mh << 32) | ml)) - (1.0 - 0x1p-53);
  const uint32_t one = ~(uint32_t)((int32_t)vh >> 31) & 0x3ff00000u;   // the high word of 1.0 in the lower half
  return fabs(t - __longlong_as_double((long long)((uint64_t)one << 32)));
}

// 1 - w for the FP32 coordinate w of U, from its upper 32 bits only: with
// s = U_hi - 2^31 as a signed 32-bit integer, the cell is c = |s| >> 8 for s >= 0
// and (|s| - 1) >> 8 for s < 0, and w = (c + 1/2) 2^-23, the midpoint of the 2^-23
// cell of the baker-transformed point (within 2^-24 of the FP64 coordinate;
// exactly its cell unless U's low 40 bits are all zero). With
// g = (signed U_hi) >> 8 this is w = 1 - |g + 1/2| 2^-23; w and 1 - w are exact in
// FP32. c24 = 2^-24, in a register that the caller keeps.
__device__ __forceinline__ float lattice_complement_f32(uint32_t hi, float c24) {
  const float g = (float)((int32_t)hi >> 8);
  float wc;
  __asm__("v_fmamk_f32 %0, %1, %2, %3" : "=v"(wc) : "v"(g), "i"(__builtin_bit_cast(uint32_t, 0x1p-23f)), "v"(c24));
  return fabsf(wc);
}

}  // namespace vecchia
