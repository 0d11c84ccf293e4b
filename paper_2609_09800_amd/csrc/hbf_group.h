// What the workgroups of one launch that wait for each other agree on; plain
// C++, so that the host can check it.
#pragma once

#include <stdint.h>

namespace hbf {

// Whether a 32-bit counter that only grows has reached `target`.  A call of
// many chunks counts past 2^32, so the two are compared by their distance,
// which stays far below 2^31 (one barrier's arrivals).
constexpr bool counter_reached(uint32_t count, uint32_t target) { return (int32_t)(count - target) >= 0; }

// A group's members are the workgroups that have started by the time it
// closes: when all `want` have, or when the first one's patience ends.  Later
// ones leave at once.  So whoever waits for a member waits for a workgroup that
// is running, also where two calls, or another stream's kernels, leave no room
// for every workgroup at the same time.
struct Member {
  uint32_t id, count;  // this workgroup's number among `count`; count 0: it came too late
};
constexpr uint32_t GROUP_CLOSED = 1u << 31;

// `w` stands for the group's two words, zero at the launch: arrive() adds 1 to
// the first and close() sets GROUP_CLOSED in it, both returning what was there;
// count() / set_count() are the second, the number of members.  wait() returns
// whether to go on waiting (only the first workgroup asks for an end).
template <typename Words>
constexpr Member group_join(Words &w, uint32_t want) {
  const uint32_t id = w.arrive();
  if (id & GROUP_CLOSED) return Member{0, 0};
  if (id + 1 == want) {  // complete (should the first one close it now, it counts the same)
    w.set_count(want);
    return Member{id, want};
  }
  uint32_t n = w.count();
  while (n == 0) {
    if (!w.wait() && id == 0) {
      n = w.close();
      w.set_count(n);
      break;
    }
    n = w.count();
  }
  return Member{id, n};
}

}  // namespace hbf
