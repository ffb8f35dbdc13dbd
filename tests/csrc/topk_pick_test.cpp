// Host check of the radix select's digit choice: the 256 threads of the last workgroup write
// the state in any order (ascending, descending, shuffled), and the k-th largest key must
// come out whatever the order, over digits with few and with many keys.
#define __host__
#define __device__
#include <algorithm>
#include <cstdio>
#include <functional>
#include <numeric>
#include <random>
#include <vector>

#include "cf_topk_pick.h"

// the k-th largest of `keys`, or the prefix that cuts off exactly k of them
static bool select(const std::vector<uint64_t> &keys, uint64_t k, int order, std::mt19937 &rng) {
  uint64_t state[6] = {0, 0, k, 0, 0, 0};
  for (int shift = 56; shift >= 0 && !state[5]; shift -= 8) {
    uint64_t own[256] = {}, at[256];
    const uint64_t prefix = state[0], mask = state[1], krem = state[2];  // read by all before any writes
    for (uint64_t key : keys)
      if ((key & mask) == prefix) ++own[(key >> shift) & 0xFF];
    uint64_t sum = 0;
    for (int d = 255; d >= 0; --d) at[d] = sum += own[d];
    std::vector<int> t(256);
    std::iota(t.begin(), t.end(), 0);
    if (order == 1) std::reverse(t.begin(), t.end());
    if (order == 2) std::shuffle(t.begin(), t.end(), rng);
    for (int d : t) cf::topk_pick(prefix, mask, krem, (uint32_t)d, shift, own[d], at[d], state);
  }
  std::vector<uint64_t> s(keys);
  std::sort(s.begin(), s.end(), std::greater<uint64_t>());
  const uint64_t n = (uint64_t)std::count_if(keys.begin(), keys.end(), [&](uint64_t q) { return q >= state[0]; });
  return n == k && s[k - 1] >= state[0] && (k == s.size() || s[k] < state[0]);
}

int main() {
  std::mt19937 rng(7);
  for (int rep = 0; rep < 60; ++rep) {
    const size_t n = 1 + rng() % 3000;
    std::vector<uint64_t> keys(n);
    const uint32_t levels = rep % 3 == 0 ? 4u : rep % 3 == 1 ? 300u : 0xFFFFFFFFu;  // ties, few ties, spread
    for (size_t i = 0; i < n; ++i) keys[i] = (uint64_t)(rng() % levels) << 32 | (0xFFFFFFFFu - (uint32_t)i);
    for (uint64_t k : {(uint64_t)1, (uint64_t)(1 + rng() % n), (uint64_t)n})
      for (int order = 0; order < 3; ++order)
        if (!select(keys, k, order, rng)) {
          std::printf("FAIL n %zu k %llu order %d levels %u\n", n, (unsigned long long)k, order, levels);
          return 1;
        }
  }
  std::printf("OK\n");
  return 0;
}
