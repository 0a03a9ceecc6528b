// Index rules of kernels that are easy to get wrong at the ends of their
// ranges, in plain C++: a test on the CPU holds them to their limits.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define FSTC_BOTH __host__ __device__
#else
#define FSTC_BOTH
#endif

namespace fstc {

// Entries that may be read from `base` on in a list of `cap` entries of which
// `count` were asked for.  Those past the list's end were refused (whoever
// reads the list learns so from a flag, which may arrive with the list).
FSTC_BOTH constexpr uint32_t list_entries(uint32_t base, uint32_t count, uint32_t cap) {
  return base >= cap ? 0u : (count < cap - base ? count : cap - base);
}

// State `lane` of the g-th 64 of V states, V where there is none.  (The lanes
// past the last state of V > 2^31 - 64 do not fit 32 bits.)
FSTC_BOTH constexpr int32_t lane_state(uint64_t g, uint32_t lane, int32_t V) {
  return g * 64 + lane < (uint64_t)V ? (int32_t)(g * 64 + lane) : V;
}

}  // namespace fstc
