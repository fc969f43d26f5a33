// The launch-shape rule over all types, rank counts and sizes from nothing to
// 2^42 bytes: a shape the configuration's limits accept, at least a row per
// wavefront and no more rows than the rule's largest tile; and the sizes where
// it changes.  Prints "ok" and exits 0 on success.
#include <cstdio>
#include <cstdlib>

#include "tuning.hpp"

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("FAIL %s:%d: %s (dtype %d ranks %d bytes %llu)\n", __FILE__, \
                  __LINE__, #c, dtype, ranks, (unsigned long long)bytes); \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

int main() {
  const int row_elems[7] = {256, 256, 512, 1024, 1024, 1024, 512};
  for (int dtype = 0; dtype < 7; ++dtype)
    for (int ranks = 1; ranks <= 16; ++ranks)
      for (int lg = -1; lg <= 42; ++lg)
        for (int d = -1; d <= 1; ++d) {
          const uint64_t bytes = lg < 0 ? 0 : (1ull << lg) + (uint64_t)d;
          const pcoll::TuneChoice c = pcoll::shape_rule(dtype, ranks, bytes);
          const int rows = c.tile_elems / row_elems[dtype];
          CHECK(c.tile_elems % 1024 == 0 && c.tile_elems >= 1024);
          CHECK(rows * row_elems[dtype] == c.tile_elems);
          CHECK(rows >= c.group_waves && rows <= 64);
          CHECK(c.group_waves >= 1 && c.group_waves <= 8);
          CHECK(c.groups_per_cu >= 1 && c.groups_per_cu <= 64);
          CHECK(c.interleave >= 0 && c.interleave <= (1 << 20));
          CHECK(c.publish_batch >= 1 && c.publish_batch <= 64);
          CHECK(c.unroll == 2 || c.unroll == 4);
        }
  // 7 and 8 ranks: tiles of 32 rows where a message has 257 to 512 of 16
  for (int dtype : {0, 1, 2, 6})
    for (int ranks : {6, 7, 8, 9, 16})
      for (uint64_t rows : {4095ull, 4096ull, 4097ull, 8191ull, 8192ull,
                            8193ull, 65536ull}) {
        const uint64_t bytes = rows * 1024;
        const int got = pcoll::shape_rule(dtype, ranks, bytes).tile_elems /
                        row_elems[dtype];
        const bool two = rows > 4096 && rows <= 8192;
        CHECK(got == (ranks <= 6 ? 32 : (ranks <= 8 && two ? 32 : 16)));
      }
  std::printf("ok\n");
  return 0;
}
