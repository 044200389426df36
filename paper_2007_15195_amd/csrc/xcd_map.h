// Blocks of a QMC launch to slots of its item list. The hardware deals
// consecutive blocks to the chip's 8 XCDs in turn (block b to XCD b mod 8), each
// with its own L2.
//  * even: many items, nearly all of one chain length of one instance, equal work.
//    Each XCD takes one contiguous eighth of the list, so that the items of one
//    term (consecutive) share an L2 for the term's rows and for the lines of their
//    partial sums (2,500 sites, m = 10, 10^4 x 10 points: 1.2% faster in FP64 and
//    0.4% in FP32 than with stripes, and 1.7% and 0.3% than with slot b).
//  * otherwise stripes of kStripe slots, so that every part of the list is spread
//    over all XCDs: a launch that several chain lengths share lists the longest
//    chains first, and instances differ in their rare steps. (With eighths one or
//    two XCDs had most of such a launch's work: 16,000 items each of 2, 4, 6, 8, 10
//    and 63 steps, 8192 points, 17.1 -> 3.4 ms; of 2, .., 10 and 30 steps 5.5 -> 1.64
//    ms; 24 uneven instances 14.0 -> 12.9 ms; 900 sites, m = 50, FP64 8.6 -> 8.3 ms.)
// The results do not depend on it.
#pragma once

#include <cstdint>

namespace vecchia {

constexpr uint32_t kXcds = 8, kStripe = 32;

// A bijection of [0, n) for any n: whole rounds of kXcds stripes (none if even), then
// the rest in kXcds contiguous parts.
__host__ __device__ __forceinline__ uint32_t xcd_slot(uint32_t b, uint32_t n, bool even) {
  const uint32_t whole = even ? 0 : n / (kXcds * kStripe) * (kXcds * kStripe);
  const uint32_t x = b % kXcds;
  if (b < whole) {
    const uint32_t j = b / kXcds;
    return (j / kStripe * kXcds + x) * kStripe + j % kStripe;
  }
  const uint32_t j = (b - whole) / kXcds, q = (n - whole) / kXcds, r = (n - whole) % kXcds;
  return whole + x * q + (x < r ? x : r) + j;
}

}  // namespace vecchia
