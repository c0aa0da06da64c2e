// Launch shapes of the rank walks (rank_plan.h).
#include "rank_plan.h"

#include <algorithm>

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
