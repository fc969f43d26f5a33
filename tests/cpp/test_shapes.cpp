// The launch-shape rule over all types, rank counts and sizes from nothing to
// 2^42 bytes: a shape the configuration's limits accept, at least a row per
// wavefront and no more rows than the rule's largest tile; and the sizes where
// it changes.  And the direct kernel's shape: every row in a tile, the grid
// within its limit, and what a caller's environment sets of it taken.  Prints
// "ok" and exits 0 on success.
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
  int ranks = 8;
  for (int dtype = 0; dtype < 7; ++dtype)
    for (uint64_t bytes : {1ull, 1024ull, 1000003ull, 1ull << 20, 1ull << 24,
                           (1ull << 31) - 7, 1ull << 36, 1ull << 40}) {
      const uint64_t span = bytes <= (1ull << 31) ? bytes : 1ull << 28;
      const uint64_t re = (uint64_t)row_elems[dtype];
      const uint64_t span_rows = (span + re - 1) / re;
      const pcoll::DirectShape d =
          pcoll::direct_shape(dtype, ranks, bytes, span, {});
      for (int tile : {0, 1, 1000, 1024, 65536, 1 << 26})
        for (int groups : {0, 1, 7, 512})
          for (int inter : {-5, -1, 0, 1, 16, 1 << 21})
            for (int waves : {-1, 0, 1, 3, 8, 9}) {
              pcoll::DirectOverride o;
              o.tile_elems = tile;
              o.groups = groups;
              o.interleave = inter;
              o.group_waves = waves;
              const pcoll::DirectShape s =
                  pcoll::direct_shape(dtype, ranks, bytes, span, o);
              const bool own = waves >= 1 && waves <= 8;
              CHECK(s.tile_rows >= 1 && s.span_tiles >= 1);
              CHECK((uint64_t)s.tile_rows * s.span_tiles >= span_rows);
              CHECK(s.groups == (bytes + span - 1) / span * s.span_tiles);
              CHECK(s.groups * 64 * (uint64_t)s.waves < (1ull << 32));
              CHECK(s.waves == (own ? waves : d.waves));
              CHECK(s.band <= (1u << 20));
              if (inter == 0 || inter == 16) CHECK((int)s.band == inter);
              if (inter < 0 || inter > (1 << 20)) CHECK(s.band == d.band);
              if (tile == 65536 && groups == 0 && span == bytes)
                CHECK(s.tile_rows == 65536 / re);
              if (groups && span == bytes) CHECK(s.groups <= (uint64_t)groups);
              if (!tile && !groups && !own)
                CHECK(s.tile_rows == d.tile_rows && s.lds == d.lds);
              else
                CHECK(s.lds == 0);
            }
    }
  std::printf("ok\n");
  return 0;
}
