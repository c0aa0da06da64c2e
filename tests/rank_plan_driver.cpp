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

// Measured walks (256 CUs, microseconds) of which one is at least a quarter
// faster: the estimates must choose it.
struct Measured {
  WalkWork work;
  FloatShape shape;
  RankShape rank;
  bool aligned;
  int64_t rows;
  double float_us, rank_us;
};
const Measured kMeasured[] = {
    {{0, 256, 9, 16, 10, 1, 621, 128, 0}, {2, 4, 1, 2, 256}, {8, 1, 4, 65280}, true, 200000, 106, 151},
    {{0, 256, 9, 16, 3, 1, 394, 128, 0}, {2, 4, 1, 2, 256}, {12, 1, 4, 59136}, true, 200000, 106, 138},
    {{0, 256, 9, 16, 1, 2, 200, 115, 0}, {2, 4, 1, 2, 256}, {8, 1, 4, 24576}, true, 1000000, 324, 456},
    {{0, 132, 9, 16, 1, 2, 166, 65, 0}, {2, 8, 2, 4, 256}, {12, 1, 4, 24576}, true, 200000, 28.9, 84.4},
    {{0, 256, 11, 16, 3, 2, 641, 128, 0}, {1, 2, 1, 1, 256}, {8, 1, 2, 61184}, true, 200000, 473, 152},
    {{0, 128, 11, 16, 3, 2, 0, 128, 0}, {1, 4, 1, 1, 256}, {8, 2, 2, 32768}, true, 1000000, 425, 135},
    {{0, 8, 11, 32, 30, 19, 52, 4, 0}, {1, 8, 2, 2, 391}, {8, 2, 2, 32768}, true, 200000, 62.6, 39.5},
    {{0, 64, 4, 144, 136, 1, 356, 0, 0}, {1, 8, 8, 144, 256}, {8, 2, 8, 32768}, true, 317161, 61.6, 87.9},
    {{0, 44, 7, 112, 100, 8, 396, 0, 0}, {1, 8, 8, 32, 256}, {8, 2, 8, 32512}, false, 398351, 176, 116},
    {{0, 44, 4, 64, 64, 1, 110, 22, 0}, {1, 8, 8, 64, 256}, {8, 2, 8, 32768}, false, 604443, 142, 75.5},
    {{0, 8, 6, 192, 184, 4, 44, 4, 0}, {1, 8, 8, 64, 512}, {8, 2, 8, 32768}, false, 809044, 236, 186},
    {{0, 136, 6, 144, 143, 5, 454, 68, 0}, {2, 8, 8, 16, 256}, {8, 2, 8, 24320}, true, 334581, 125, 156},
    {{0, 116, 7, 864, 856, 40, 1160, 0, 0}, {2, 8, 8, 16, 256}, {8, 1, 8, 40704}, true, 314738, 517, 661},
    {{0, 120, 6, 112, 110, 3, 369, 60, 0}, {2, 8, 8, 32, 256}, {8, 2, 8, 30464}, true, 448862, 98.4, 142},
    {{0, 206, 4, 96, 94, 1, 342, 103, 0}, {2, 4, 8, 64, 256}, {8, 2, 8, 24320}, false, 233218, 461, 108},
    {{0, 84, 7, 144, 134, 7, 672, 0, 0}, {2, 8, 8, 16, 256}, {8, 2, 8, 32768}, false, 3229145, 2.24e+03, 1.12e+03},
    {{0, 148, 5, 128, 128, 3, 381, 74, 0}, {2, 8, 8, 16, 256}, {8, 2, 8, 20224}, false, 3619389, 3.94e+03, 1.24e+03},
    {{0, 100, 4, 144, 140, 1, 245, 50, 0}, {2, 8, 8, 128, 256}, {8, 2, 8, 32768}, false, 3293471, 2.27e+03, 721},
    {{0, 184, 7, 144, 141, 4, 644, 92, 0}, {2, 4, 4, 8, 256}, {12, 1, 8, 49920}, false, 270664, 545, 184},
    {{0, 43, 5, 64, 64, 1, 132, 21, 0}, {1, 8, 8, 64, 256}, {8, 2, 8, 32768}, false, 302877, 85, 52.2},
    {{0, 6, 6, 16, 12, 1, 45, 0, 0}, {1, 8, 8, 16, 631}, {8, 2, 8, 32768}, false, 322568, 14.9, 21},
    {{0, 16, 4, 16, 11, 1, 61, 0, 0}, {1, 8, 8, 16, 1024}, {8, 2, 8, 32768}, true, 1617499, 46.9, 61},
    {{0, 40, 7, 16, 13, 1, 118, 20, 0}, {1, 8, 8, 16, 256}, {8, 2, 8, 32768}, false, 2562151, 494, 206},
    {{0, 58, 4, 16, 13, 1, 129, 4, 0}, {1, 8, 8, 16, 256}, {8, 2, 8, 32768}, false, 1211985, 328, 146},
    {{1, 40, 3, 1, 5, 2, 11, 11, 18}, {1, 8, 1, 1, 256}, {12, 2, 1, 24576}, true, 300000, 20.7, 46},
    {{1, 31, 3, 1, 10, 2, 21, 17, 38.5}, {1, 8, 1, 1, 256}, {12, 2, 1, 24576}, true, 319540, 30.3, 46.6},
    {{1, 248, 3, 1, 5, 2, 10, 22, 19.8}, {1, 2, 1, 1, 256}, {12, 2, 1, 24576}, true, 888065, 364, 539},
    {{1, 200, 2, 1, 5, 2, 6, 9, 15}, {1, 2, 1, 1, 256}, {12, 2, 1, 24576}, true, 300000, 79, 157},
    {{1, 176, 3, 1, 17, 1, 0, 72, 62.8}, {1, 2, 1, 1, 256}, {16, 1, 1, 24576}, false, 433859, 1.02e+03, 120},
    {{1, 218, 3, 1, 20, 2, 99, 10, 72}, {1, 2, 1, 1, 256}, {16, 1, 1, 24576}, false, 211932, 341, 89.1},
    {{1, 36, 14, 1, 17, 2, 90, 18, 82.9}, {1, 8, 1, 1, 256}, {12, 2, 1, 24576}, true, 1680309, 158, 225},
    {{1, 6, 14, 1, 7, 2, 18, 3, 32.2}, {1, 8, 1, 1, 768}, {12, 2, 1, 24576}, false, 653619, 35.1, 52},
    {{1, 128, 9, 1, 5, 2, 90, 56, 24.5}, {2, 8, 2, 1, 256}, {16, 1, 1, 24576}, true, 1500000, 175, 254},
    {{1, 128, 14, 1, 20, 2, 224, 64, 95.3}, {2, 8, 2, 1, 256}, {12, 1, 1, 24576}, true, 300000, 64, 99.3},
    {{1, 252, 8, 1, 31, 2, 339, 126, 159.6}, {1, 2, 1, 1, 256}, {8, 1, 1, 24576}, false, 1386500, 4.81e+03, 917},
    {{1, 88, 8, 1, 7, 2, 93, 44, 36.2}, {2, 8, 2, 1, 256}, {16, 1, 1, 24576}, false, 1605683, 827, 311},
    {{1, 216, 8, 7, 227, 8, 629, 108, 1111.5}, {1, 2, 1, 1, 256}, {8, 1, 1, 24576}, true, 237925, 997, 315},
    {{1, 200, 14, 4, 100, 5, 533, 100, 516.3}, {1, 2, 1, 1, 256}, {8, 1, 1, 24576}, true, 1500000, 3.11e+03, 1.19e+03},
};

void check_estimates() {
  for (const Measured &m : kMeasured) {
    const RowKind kind = row_kind(m.aligned, m.work.features);
    const double f = float_walk_us(m.work, m.shape, kind, (double)m.rows, 256);
    const double r = rank_walk_us(m.work, m.rank, kind, (double)m.rows, 256);
    if ((r < f) != (m.rank_us < m.float_us)) {
      fprintf(stderr, "%d trees of depth %d over %d features, %lld rows: estimated %g and %g us, "
              "measured %g and %g\n", m.work.trees, m.work.depth, m.work.features,
              (long long)m.rows, f, r, m.float_us, m.rank_us);
      exit(1);
    }
  }
}

int main() {
  check_estimates();
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
