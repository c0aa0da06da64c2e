// Launch shapes of the rank walks (rank_plan.h).
#include "rank_plan.h"

#include <algorithm>
#include <cmath>

namespace ml2 {
namespace {

constexpr int kLanes = 64;
constexpr uint32_t kMaxSlot = 64 * 1024;

struct Waves {
  int waves, per_cu;
};

// The register class of a kernel that shares a CU with `total` waves in all.
int wave_class(int total) { return total > 16 ? 24 : total > 12 ? 16 : total > 8 ? 12 : total > 4 ? 8 : 4; }

// Bytes that the staging registers of `waves` waves of a class hold.
size_t stage_bytes(int cls, int waves) {
  return (size_t)rank_stage_regs(cls) * 16 * kLanes * waves;
}

size_t queue_bytes(int waves) { return (size_t)waves * 2 * kLanes * sizeof(int32_t); }

uint32_t past_tile(uint32_t tile) {
  uint32_t past = kRankRow;
  while (past < tile) past *= 2;
  return past;
}

size_t ragged_lds(uint32_t tile, int waves) {
  // a leaf reads a code within rank_ragged_mask of its lane's column
  const size_t fixed = kRaggedChunkBytes + (size_t)waves * tile;
  return std::max(fixed + queue_bytes(waves) + waves * sizeof(int),
                  fixed - tile + kRankRow + past_tile(tile));
}

}  // namespace

// Two workgroups of eight waves first: one walks while the other waits at a
// barrier or for its rows (16M x 128 validity 7.20 -> 6.76 ms against one of
// sixteen).  They need room for a slot of two groups of trees each, or of 32
// KiB (a shorter one spends the gain on restaging: 4M x 96, depth 8, 24 KiB
// slots: 3.83 ms, one workgroup of sixteen waves with 55 KiB: 3.64); else one
// workgroup of as many waves as leave that room, by fours, as each SIMD takes
// a fourth (16M x 128 performance: twelve waves and a 58 KiB slot 14.5 ms,
// sixteen and 23 KiB 16.7, ten 16.4, eight 16.6).  Tiles of 256 features (32
// KiB per wave) leave three waves at least.
bool rank_shape(uint32_t tile, int D, RankShape *out) {
  if (D < kRankMinDepth || D > kRankMaxDepth) return false;
  const Waves shapes[] = {{8, 2}, {16, 1}, {12, 1}, {8, 1}, {7, 1},
                          {6, 1}, {5, 1},  {4, 1},  {3, 1}};
  const uint32_t one = (uint32_t)kRankGroup[D] * rank_tree_bytes(D);
  const uint32_t need = std::max(one, std::min<uint32_t>(2 * one, 32 * 1024));
  for (const Waves &sh : shapes) {
    const size_t fixed = (size_t)sh.waves * tile + queue_bytes(sh.waves);
    const size_t lds = kLdsBudget / sh.per_cu;
    if (fixed >= lds) continue;
    const uint32_t slot =
        (uint32_t)std::min({lds - fixed, (size_t)kMaxSlot,
                            stage_bytes(wave_class(sh.waves * sh.per_cu), sh.waves)}) & ~255u;
    if (slot < need) continue;
    *out = RankShape{sh.waves, sh.per_cu, kRankGroup[D], slot};
    return true;
  }
  return false;
}

// The slot is fixed.  The walk is bound by the latency of its chain of reads,
// so as many waves as fit, two workgroups of twelve first (16M x 128 round,
// 300 trees of depth up to 14 over 64 features: 8 waves per CU 9.2 ms, 12 6.6,
// 16 5.4, 24 4.6).
bool rank_ragged_shape(uint32_t tile, RankShape *out) {
  const Waves shapes[] = {{12, 2}, {16, 1}, {12, 1}, {8, 1}, {4, 1}};  // (four hold any tile)
  for (const Waves &sh : shapes) {
    if (ragged_lds(tile, sh.waves) * sh.per_cu > kLdsBudget) continue;
    *out = RankShape{sh.waves, sh.per_cu, 1, kRaggedChunkBytes};
    return true;
  }
  return false;
}

RowKind row_kind(bool aligned, int32_t features) {
  if (!aligned) return kRowsSingle;
  return features % 4 == 0 && features <= 128 ? kRowsAhead : kRowsVector;
}

// The estimates are linear in what a walk does, fitted (least squares of the
// relative error) to both walks' times over 9,200 shapes without a mask:
// perfect trees of depth 4 to 12 and ragged ones of depth 1 to 14, 1 to 1,500
// trees, 4 to 256 features in aligned and unaligned rows, 100,000 to 4 million
// rows, 256 CUs.  Median error 6 to 10 %.  Of the 7,300 large enough to rank
// (rank_takes), the walk taken with them is more than 5 % slower than the float
// walk for 3 %, and for 8 % without them.
double float_walk_us(const WalkWork &w, const FloatShape &s, RowKind kind, double rows, int cus) {
  struct Fit {
    double call, row[3], chunk, round, visit, chain;
  };
  static const Fit fits[2][2] = {
      // one lane per candidate, two; perfect trees, ragged ones
      {{3.3, {0.0106, 0.0129, 0.0394}, 0.62, 0.0, 0.00239, 0.0525},
       {0.0, {0.0025, 0.0066, 0.0717}, 0.44, 2.80, 0.00271, 0.0310}},
      {{5.7, {0.0117, 0.0168, 0.0418}, 3.14, 0.0, 0.00895, 0.0193},
       {1.9, {0.0077, 0.0109, 0.0672}, 6.98, 1.56, 0.00789, 0.0}}};
  const Fit &c = fits[w.ragged != 0][s.split == 2];
  const double rounds = std::max(1.0, std::ceil(rows / (64.0 * s.waves / s.split * s.grid)));
  const double per_cu = std::ceil((double)s.grid / cus);
  const double lanes = s.waves * per_cu / s.split;
  const int chunks = (w.records + s.chunk - 1) / s.chunk;
  const double visits = w.ragged ? w.path : (double)w.records * w.depth;
  const double chain = visits / s.split / (w.ragged ? 1 : s.group);
  // (copies: about 3,500 bytes per wave and microsecond)
  const double chunk =
      s.copied ? (double)s.chunk * record_bytes(w.ragged ? 0 : w.depth) / (3500.0 * s.waves)
               : c.chunk;
  return c.call + rounds * (w.features * lanes * c.row[kind] +
                            (chunks > 1 ? chunks * per_cu * chunk : 0.0) + c.round +
                            visits * lanes * c.visit + chain * c.chain);
}

double rank_walk_us(const WalkWork &w, const RankShape &s, RowKind kind, double rows, int cus) {
  const double rounds = std::max(1.0, std::ceil(rows / (64.0 * s.waves * s.per_cu * cus)));
  const double u = rows / (cus * 3906.25);  // a million rows on 256 CUs
  const double lines = (w.features + kRankLine - 1) / kRankLine;
  const bool whole = kind != kRowsSingle && w.features % 4 == 0;
  if (w.ragged)
    return 3.1 + rounds * (w.steps * 0.019 + w.path * 0.051 + w.slots * 2.7) +
           u * (lines * (whole ? 21.2 : 28.0) + w.steps * 0.128 + w.path * 0.124);
  const int top = std::min(w.depth, 5);
  return 5.3 +
         rounds * (lines * 2.36 + w.steps * 0.035 +
                   (double)w.trees * w.depth / kRankGroup[w.depth] * 0.053 + w.slots * 0.59) +
         u * (lines * (whole ? 4.23 : 10.8) + w.steps * 0.013 + w.grids * 0.038 +
              (double)w.trees * (top * 0.118 + (w.depth - top) * 0.154));
}

uint32_t rank_ragged_mask(uint32_t tile, RankMode mode) {
  return (past_tile(tile) - 1) & (mode == kRankByte ? ~0xFCu : ~0xFDu);
}

// As many workgroups as the chip holds or the pool has units of 64 rows, of no
// more waves than a workgroup has units.
RankLaunch rank_launch(const RankShape &shape, uint32_t tile, bool ragged, int64_t units,
                       int cu_count, bool perf) {
  int w = shape.waves, per_cu = shape.per_cu;
  if (units <= (int64_t)cu_count * 8) per_cu = 1;
  for (int less : {12, 8, 4})
    if (less < w && units <= (int64_t)cu_count * per_cu * less) w = less;
  RankLaunch l{};
  l.waves = w;
  l.per_cu = per_cu;
  l.cls = wave_class(w * per_cu);
  l.lds = ragged ? ragged_lds(tile, w)
                 : (size_t)w * tile + shape.slot_bytes + (perf ? queue_bytes(w) : 0);
  l.grid = (int32_t)std::max<int64_t>(1, std::min<int64_t>(units, (int64_t)cu_count * per_cu));
  return l;
}

bool rank_stages_slot(const RankShape &shape, bool ragged, const RankLaunch &l) {
  const int regs = ragged ? rank_ragged_stage_regs(l.cls) : rank_stage_regs(l.cls);
  return (size_t)regs * 16 * kLanes * l.waves >= shape.slot_bytes && l.lds <= kLdsBudget;
}

}  // namespace ml2
