// Launch shapes of the rank walks checked on the host: for every tile (1 to
// 128 rows of codes, the most 256 features take) and depth, a shape exists,
// its slot holds a group of trees, and every launch over it, from one unit of
// rows to more than the chip holds, stages the whole slot within the LDS and
// the kernel's launch bounds.
#include <stdio.h>
#include <stdlib.h>

#include "rank_plan.h"

using namespace ml2;

#define CHECK(c)                                                                           \
  do {                                                                                     \
    if (!(c)) {                                                                            \
      fprintf(stderr, "%s:%d: %s (tile %u, depth %d)\n", __FILE__, __LINE__, #c, tile, D); \
      exit(1);                                                                             \
    }                                                                                      \
  } while (0)

static void check_launches(const RankShape &s, uint32_t tile, int D, bool ragged) {
  for (int cus : {1, 32, 256, 304})
    for (bool perf : {false, true})
      for (int64_t per_cu = 0; per_cu <= 40; ++per_cu)
        for (int64_t units : {per_cu * cus, per_cu * cus + 1}) {
          if (units < 1) continue;
          const RankLaunch l = rank_launch(s, tile, ragged, units, cus, perf);
          CHECK(l.waves >= 1 && l.waves <= s.waves && l.per_cu >= 1 && l.per_cu <= s.per_cu);
          CHECK(l.waves * l.per_cu <= l.cls);
          CHECK(l.waves <= (ragged && l.cls == 24 ? 12 : l.cls));  // __launch_bounds__
          CHECK(l.cls == 4 || l.cls == 8 || l.cls == 12 || l.cls == 16 || (ragged && l.cls == 24));
          CHECK(rank_stages_slot(s, ragged, l));
          CHECK(l.lds * l.per_cu <= kLdsBudget);
          CHECK(l.grid >= 1 && l.grid <= units && l.grid <= cus * l.per_cu);
        }
}

int main() {
  for (int rows = 1; rows <= 128; ++rows) {
    const uint32_t tile = (uint32_t)rows * kRankRow;
    for (int D = kRankMinDepth; D <= kRankMaxDepth; ++D) {
      RankShape s{};
      CHECK(rank_shape(tile, D, &s));
      CHECK(s.group == kRankGroup[D] && s.slot_bytes % 256 == 0);
      CHECK(s.slot_bytes >= (uint32_t)s.group * rank_tree_bytes(D));
      check_launches(s, tile, D, false);
    }
    const int D = 0;
    RankShape s{};
    CHECK(rank_ragged_shape(tile, &s));
    check_launches(s, tile, D, true);
    // a leaf's read: any offset under the mask, from the last wave's tile
    for (RankMode mode : {kRankByte, kRankHalf}) {
      const uint32_t mask = rank_ragged_mask(tile, mode);
      CHECK((mask & 0xFFu) == (mode == kRankByte ? 3u : 2u));
      CHECK(mask + 4u >= tile - kRankRow);
      const RankLaunch l = rank_launch(s, tile, true, 1 << 20, 256, false);
      CHECK(s.slot_bytes + (uint32_t)l.waves * tile - tile + 252u + mask + 2u <= l.lds);
    }
  }
  printf("ok\n");
  return 0;
}
