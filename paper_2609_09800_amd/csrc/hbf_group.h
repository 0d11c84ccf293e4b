// What the workgroups of one launch that wait for each other agree on; plain
// C++, so that the host can check it.
#pragma once

#include <stdint.h>

namespace hbf {

// Whether a 32-bit counter that only grows has reached `target`.  A call of
// many chunks counts past 2^32, so the two are compared by their distance,
// which stays far below 2^31 (one barrier's arrivals).
constexpr bool counter_reached(uint32_t count, uint32_t target) { return (int32_t)(count - target) >= 0; }

}  // namespace hbf
