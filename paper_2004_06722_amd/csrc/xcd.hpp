#pragma once
// Order of the work-groups over the chip's eight dies (XCDs).

#include <cstdint>
#include <hip/hip_runtime.h>

namespace bp {

// Work-groups reach the XCDs round-robin, each with an L2 of its own, so
// neighbours in blockIdx never share one. A kernel that reads through a map,
// and whose neighbours read parts of the same 128-byte lines, takes its work
// in the order of this bijection of [0, nb): each XCD gets RUN consecutive
// blocks out of every 8 RUN (the last, incomplete 8 RUN keep their order). Long
// runs are slower again: eighths of the whole range lie far apart in memory,
// and neighbours that scatter atomically at the same time contend.
// Gathers and mass, 20 iterations (runs of 16 to 128 alike, 4 and 8 up to 2%
// slower): p = 6, 41x37x29 elements 4.92 -> 4.49 ms; p = 2, 100x90x80 6.95 ->
// 6.16 ms. Collocated stiffness, with its interior nodes in blocks of their
// own (4, 16, 32, 64 tried): p = 7, E = 16x16x8, 60 iterations 2.05 -> 2.01 ms,
// E = 64^3 55.4 -> 55.0 ms; three components, E = 32^3 16.2 -> 16.0 ms (runs of
// 4 and 16: 16.4 to 16.6). Gauss-Legendre stiffness (kXcdRunGL; 4, 8, 16, 32
// tried): p = 7, E = 48^3 29.1 -> 27.8 ms (8: 28.0, 4: 28.3, 32: 28.1).
constexpr uint32_t kXcdRun = 32, kXcdRunGL = 16;
template <uint32_t RUN = kXcdRun>
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t nb) {
  constexpr uint32_t G = 8 * RUN;
  const uint32_t g = b / G, r = b % G;
  return b - r + G <= nb ? g * G + (r % 8) * RUN + r / 8 : b;
}

}  // namespace bp
