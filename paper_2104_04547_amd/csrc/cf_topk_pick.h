// The digit choice of the radix select (cf_select.hip), shared with its host test.
#pragma once

#include <stdint.h>

namespace cf {

// Select state: [0] prefix, [1] mask of decided bits, [2] k remaining, [3] collected count,
// [5] 1 when the prefix already cuts off exactly k keys ([4] is free).
//
// One thread per digit: `own` keys under the prefix have it, `at` have it or a larger one.
// The one thread whose digit holds the k-th largest key writes the state.  prefix, mask and
// krem are what state[0 .. 2] held before the pass: every thread has read them before a
// barrier, since a read beside the write could find the count already reduced and choose a
// second digit.
__host__ __device__ inline void topk_pick(uint64_t prefix, uint64_t mask, uint64_t krem, uint32_t digit, int shift,
                                          uint64_t own, uint64_t at, uint64_t *state) {
  const uint64_t above = at - own;  // keys with a larger digit
  if (above < krem && at >= krem) {
    state[0] = prefix | (uint64_t)digit << shift;
    state[1] = mask | (uint64_t)0xFF << shift;
    state[2] = krem - above;
    state[5] = krem - above == own ? 1 : 0;  // the whole bucket: no key below it has to be told apart
  }
}

}  // namespace cf
