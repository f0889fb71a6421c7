#pragma once
// Order of the work-groups over the chip's eight dies (XCDs).

#include <cstdint>
#include <hip/hip_runtime.h>

namespace bp {

// Work-groups reach the XCDs round-robin, each with an L2 of its own, so
// neighbours in blockIdx never share one. A kernel that reads through a map,
// and whose neighbours read parts of the same 128-byte lines, takes its work
// in the order of this bijection of [0, nb): each XCD gets kXcdRun consecutive
// blocks out of every 8 kXcdRun (the last, incomplete 8 kXcdRun keep their
// order). For kernels that gather and write plainly: with an atomic scatter
// neighbours on one XCD contend for the lines they share, and the stiffness
// kernels are faster round-robin. Runs of 16 to 128 measured alike, 4 and 8
// up to 2% slower. Mass solve, p = 6, 41x37x29 elements, 20 iterations:
// 4.88 -> 4.48 ms; p = 2, 100x90x80: 6.96 -> 6.14 ms.
constexpr uint32_t kXcdRun = 32;
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t nb) {
  constexpr uint32_t G = 8 * kXcdRun;
  const uint32_t g = b / G, r = b % G;
  return b - r + G <= nb ? g * G + (r % 8) * kXcdRun + r / 8 : b;
}

}  // namespace bp
