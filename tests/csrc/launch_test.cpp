// Host check of the launch sizes: every count of items gives at least one workgroup and
// fewer than 2^32 threads, and small counts one workgroup per item.
#include <cstdio>
#include <initializer_list>

#include "cf_launch.h"

int main() {
  const int64_t limit = (int64_t)1 << 32;
  for (int64_t items : {(int64_t)0, (int64_t)1, (int64_t)2, (int64_t)1000, (int64_t)1 << 20, ((int64_t)1 << 20) + 1,
                        (int64_t)1 << 24, ((int64_t)1 << 31) / 32, (int64_t)1 << 31, (int64_t)1 << 40}) {
    const int64_t g = cf::item_groups(items);
    if (g < 1 || g > (items < 1 ? 1 : items) || g * 1024 >= limit || (items >= 1 && items <= 1 << 20 && g != items)) {
      std::printf("FAIL %lld -> %lld\n", (long long)items, (long long)g);
      return 1;
    }
  }
  std::printf("OK\n");
  return 0;
}
