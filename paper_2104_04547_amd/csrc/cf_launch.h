// Sizes of launches whose work items may be many (host side, no HIP types).
#pragma once

#include <stdint.h>

namespace cf {

// Workgroups for `items` work items that they take in a grid-stride loop.  A launch of
// 2^32 threads or more is cut off without an error, so the count is capped: 2^20
// workgroups of up to 1024 threads, a thousand rounds of the chip.
inline unsigned item_groups(int64_t items) {
  constexpr int64_t kMost = 1 << 20;
  return (unsigned)(items < 1 ? 1 : items < kMost ? items : kMost);
}

}  // namespace cf
