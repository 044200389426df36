// Blocks of a QMC launch to slots of its item list. The hardware deals
// consecutive blocks to the chip's 8 XCDs in turn (block b to XCD b mod 8), each
// with its own L2. Slots go to the XCDs in stripes of kStripe consecutive ones, so
// that the items of one term (consecutive) mostly share an L2 for the term's rows
// and for the lines of their partial sums, and so that every part of the list is
// spread over all XCDs: a launch that several chain lengths share lists the longest
// chains first. (One contiguous eighth of the list per XCD left such a launch's
// work to one or two of them: 16,000 items each of 2, 4, 6, 8, 10 and 63 steps,
// 8192 points, 17.1 -> 3.4 ms; of 2, .., 10 and 30 steps 5.5 -> 1.64 ms; for a
// launch of one length the two measure the same.) The results do not depend on it.
#pragma once

#include <cstdint>

namespace vecchia {

constexpr uint32_t kXcds = 8, kStripe = 32;

// A bijection of [0, n) for any n: whole rounds of kXcds stripes, then the rest in
// kXcds contiguous parts.
__host__ __device__ __forceinline__ uint32_t xcd_slot(uint32_t b, uint32_t n) {
  const uint32_t whole = n / (kXcds * kStripe) * (kXcds * kStripe);
  const uint32_t x = b % kXcds;
  if (b < whole) {
    const uint32_t j = b / kXcds;
    return (j / kStripe * kXcds + x) * kStripe + j % kStripe;
  }
  const uint32_t j = (b - whole) / kXcds, q = (n - whole) / kXcds, r = (n - whole) % kXcds;
  return whole + x * q + (x < r ? x : r) + j;
}

}  // namespace vecchia
